// Host side of libdeer: context, buffer carving, call-order state machine, kernel launches.
// The C ABI is declared in include/deer.h.  Nothing here allocates device memory.
#include "deer_kernels.hpp"
#include "deer_block.hpp"
#include "deer_stream.hpp"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "deer.h"

using namespace deer;

// Scratch of deer_accept_and_commit_static, the entry point that allocates nothing: the per-share candidates of the
// sampling acceptance kernel (ACC_NB entries per sequence) followed by one arrival counter per sequence.  Every GPU
// the library runs on holds its own copy until the process ends.
constexpr int STATIC_MAX_BATCH = 64;
constexpr size_t STATIC_PART_BYTES = (size_t)STATIC_MAX_BATCH * ACC_NB * sizeof(AccPart);
constexpr size_t STATIC_SCRATCH_BYTES = STATIC_PART_BYTES + (size_t)STATIC_MAX_BATCH * sizeof(int);
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];
// The array's name is a host-side stand-in, not a device address: host code uses the address that
// hipGetSymbolAddress gives, resolved once per device (with that device current) by deer_init_models.
constexpr int MAX_DEVICES = 64;
static void *g_scratch_ptr[MAX_DEVICES] = {};

namespace {

thread_local std::string g_init_error;


constexpr int STAMP_MAX_BLOCKS = 4096;   // workgroups whose stamps deer_debug_gemm_stamps can record (8 stamps each)
constexpr int PREFILL_TILES = 128;   // row tiles that a prefill pass may have at any batch size (4096 rows: every pass streams the weights once)
constexpr int PART_TILES_MIN = 16;   // split-K partials exist for passes of up to max(2 * batch, 16) row tiles
constexpr int MAX_NS = 32;          // key-range splits of block attention
constexpr size_t H_UP_MAX = 1 << 20;  // most page-locked host memory of a context for uploads
constexpr int LM_TILES = 2, LM_COLS = 256 * 128;   // LM heads of up to so many row tiles and more columns run in k_lm_head
constexpr int SLIM_MAX_D = 4096, SLIM_TILES = 4;   // passes of up to 4 row tiles of a model up to this width may use k_gemm_slim (64 sums of squares per row)
constexpr int NARROW_MAX_D = 1024;  // residual width up to which a dense model's O projection runs in 32-column workgroups
constexpr int NEXT_SPAN_BYTES = 16 << 10;      // fetched ahead per 32-column block of a next-launch workgroup (4 blocks: 8 loads per thread)
constexpr int KV_FETCH_MAX_BYTES = 1 << 20;    // fetched ahead per kv head of K and of V^T: a share of one XCD's 4 MB L2
constexpr int ATT_HEAD_MAX_TILES = 12;   // per-head attention: most key tiles one wave may have to go through (equal or better up to 9, measured)
constexpr size_t PART_COLS = 131072; // fp32 columns of split-K partials per row (S * N <= PART_COLS)

size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

struct ModelRT {
    deer_model_cfg c{};
    int n_qkv = 0, kattn = 0, F = 0;   // fused QKV width, Hq*hd, FFN width used by GEMMs
    int ssq_sub = 1;   // passes of many row tiles: sums of squares of the residual stream per 128-column group (1) or per 32-column block (4)
    // weights (device)
    char *w = nullptr;
    size_t off_embed = 0, off_lm = 0, off_layers = 0, layer_bytes = 0;
    size_t lo_qkv = 0, lo_o = 0, lo_gu = 0, lo_d = 0;   // offsets inside a layer (gu/d: expert 0 for a mixture)
    size_t lo_router = 0, exp_gu_bytes = 0, exp_d_bytes = 0;   // mixture: router, per-expert matrix sizes
    size_t weight_bytes = 0;
    // kv (device, elements of bf16)
    uint16_t *kv = nullptr;
    size_t kv_k_base = 0, kv_v_base = 0, kv_layer_stride = 0, kv_seq_stride = 0, kv_head_stride = 0;
    size_t kv_bytes = 0;
    double *theta = nullptr;           // device [hd/2]
};

// What a pass writes on its way.  A second set lets the drafter's prefill run beside the target's (see enqueue_prefill).
struct PassBufs {
    RowMeta rm{};
    float2 *cs = nullptr;
    float *h = nullptr, *ssq = nullptr, *part = nullptr, *opart = nullptr;
    uint4 *xa_hi = nullptr, *xa_lo = nullptr, *xb_hi = nullptr, *xb_lo = nullptr, *q_hi = nullptr, *q_lo = nullptr;
    int *gemm_cnt = nullptr, *attn_cnt = nullptr;   // arrival counters, zero between kernels
    size_t part_floats = 0;   // capacity of `part`
};

struct Work : PassBufs {   // carved from the workspace
    PassBufs beside;
    SeqState st{};
    float *logits[2] = {nullptr, nullptr};
    RowStat *stat = nullptr;
    RowResult *res[2] = {nullptr, nullptr};
    AcceptOut ao{};
    int *ids = nullptr;                // prompt staging [max_seq]
    // mixture-of-experts routing and staging (target only)
    int *route_e = nullptr, *pairs = nullptr;
    int4 *items = nullptr;
    float *route_w = nullptr, *moe_out = nullptr;
    unsigned long long *moe_touched = nullptr;   // (layer, expert) pairs streamed since the last read
    uint4 *act_hi = nullptr, *act_lo = nullptr, *xg_hi = nullptr, *xg_lo = nullptr;   // per expert: FFN activations, gathered input rows
    size_t cnt_bytes = 0; char *cnt_base = nullptr;
    double *theta[2] = {nullptr, nullptr};
    AccPart *acc_part = nullptr; int *acc_cnt = nullptr;   // sampling acceptance: per-share candidates, arrival counters
    int4 *pf_desc[2] = {nullptr, nullptr};   // prefill, per model: the pass's attention tiles (see PassRows)
    char *up = nullptr;       // start of the block that the host uploads; offsets of the descriptors and the prompts in it
    size_t up_desc = 0, up_ids = 0;
    unsigned long long *stamps = nullptr;   // [STAMP_MAX_BLOCKS][8], written on request (deer_debug_gemm_stamps)
    size_t bytes = 0;
};

enum State { ST_INIT = 0, ST_PREFILLED, ST_DRAFTED, ST_VERIFIED };

}  // namespace

struct deer_ctx {
    deer_init_params p{};
    ModelRT m[2];
    Work wk;
    hipStream_t stream = nullptr;
    hipStream_t side = nullptr;      // the drafter's prefill passes, between the two events; null: none could be made
    hipEvent_t fork = nullptr, join = nullptr;
    State state = ST_INIT;
    int batch = 0;
    int cur_k = 0;
    float cur_T = 0.f;
    int max_tiles = 0;
    int block_gemm = 128;            // deer_debug_gemm_tiled: 0 never blocked; 128 where it is estimated to be faster; less: from 8 row tiles on
    int force_nb = 0, force_ring = 0, force_S = 0;   // deer_debug_gemm_block; force_nb 0: off
    // deer_debug_gemm_stamps: which streaming-GEMM launch of which model's passes records its stamps
    int stamp_model = 0, stamp_launch = -1, stamp_blocks = 0, gemm_launch_idx = 0, cur_pass_model = 0;
    bool slim = true;                // deer_debug_gemm_tiled: off where it asks for the plain streaming kernels
    int route_spread = 0;            // deer_debug_route_spread: synthetic uniform routing for mixture models
    int bonus = 0;                   // 1: verify k + 1 rows, commit one more target token after k accepted drafts
    void *static_scratch = nullptr;  // this device's copy of `scratch`
    const int *wk_draft = nullptr;   // draft buffer of the last verify_block
    std::vector<int> h_len, h_ing_n, h_finished;
    std::vector<char> h_ao;          // host staging of the acceptance results (pageable; used only if pinning failed)
    char *h_pin = nullptr;           // the same, page-locked: the copy lands without an intermediate staging copy
    size_t h_pin_bytes = 0;
    char *h_pin_dev = nullptr;       // its device address: the acceptance kernels write their results there
    char *h_up = nullptr;            // page-locked image of what the host uploads (prompts beyond it: h_up_vec)
    size_t h_up_bytes = 0;
    std::vector<char> h_up_vec;
    std::string err;
    // optional per-launch timing (deer_debug_profile)
    bool prof_on = false;
    struct ProfRec { int cls; hipEvent_t a, b; double bytes; int launches; };
    std::vector<ProfRec> prof;
    int prof_open_cls = -1;          // a run of consecutive launches of one class is being timed
    hipEvent_t prof_open_a = nullptr;
    double prof_open_bytes = 0.0;
    int prof_open_launches = 0;
    std::vector<hipEvent_t> ev_pool;
    size_t ev_used = 0;
};

namespace {

int fail(deer_ctx *c, int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (c) c->err = buf; else g_init_error = buf;
    return code;
}

hipEvent_t prof_event(deer_ctx *c) {
    if (c->ev_used == c->ev_pool.size()) {
        hipEvent_t e = nullptr;
        if (hipEventCreate(&e) != hipSuccess) return nullptr;
        c->ev_pool.push_back(e);
    }
    return c->ev_pool[c->ev_used++];
}

// Timing of launches when profiling is on.  Launches of one class that follow each other directly on the stream (the
// O, gate/up and down projections and the next layer's QKV projection) share one pair of events: an event between
// two of them costs more than the gap it would measure.  prof_close() ends the run that is open; it is called before
// a launch of another class, before every launch that is not timed, and before the records are read.
void prof_close(deer_ctx *c) {
    if (c->prof_open_cls < 0) return;
    hipEvent_t b = prof_event(c);
    if (b) {
        (void)hipEventRecord(b, c->stream);
        c->prof.push_back({c->prof_open_cls, c->prof_open_a, b, c->prof_open_bytes, c->prof_open_launches});
    }
    c->prof_open_cls = -1;
}
struct ProfScope {
    ProfScope(deer_ctx *c, int cls, double bytes) {
        if (!c->prof_on) return;
        if (c->prof_open_cls != cls) {
            prof_close(c);
            hipEvent_t a = prof_event(c);
            if (!a) return;
            (void)hipEventRecord(a, c->stream);
            c->prof_open_cls = cls; c->prof_open_a = a; c->prof_open_bytes = 0.0; c->prof_open_launches = 0;
        }
        c->prof_open_bytes += bytes;
        c->prof_open_launches += 1;
    }
};

#define HIPCHK(c, expr)                                                                            \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess) return fail((c), DEER_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

#define LAUNCHCHK(c, name)                                                                          \
    do {                                                                                            \
        hipError_t e_ = hipGetLastError();                                                          \
        if (e_ != hipSuccess) return fail((c), DEER_EHIP, "launch %s: %s", name, hipGetErrorString(e_)); \
    } while (0)

const char *check_model(const deer_model_cfg &c) {
    if (c.n_layers < 1 || c.d_model < 128 || c.vocab < 128) return "n_layers/d_model/vocab too small";
    if (c.head_dim != 32 && c.head_dim != 64 && c.head_dim != 128) return "head_dim must be 32, 64 or 128";
    if (c.n_kv_heads < 1 || c.n_q_heads % c.n_kv_heads) return "n_q_heads must be a multiple of n_kv_heads";
    if (c.d_model % CG) return "d_model must be a multiple of 128";
    if (c.d_model > 8192) return "d_model above 8192 is not supported (64 column groups of sums of squares per row)";
    if (((c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim) % CG) return "fused QKV width must be a multiple of 128";
    if ((c.n_q_heads * c.head_dim) % 16) return "n_q_heads*head_dim must be a multiple of 16";
    if (c.vocab % CG) return "vocab must be a multiple of 128";
    if (c.n_experts) {
        if (c.n_experts > 128 || c.top_k < 1 || c.top_k > 8 || c.top_k > c.n_experts) return "mixture needs n_experts <= 128 and 1 <= top_k <= 8";
        if (c.d_ff_expert < 64 || c.d_ff_expert % 64) return "d_ff_expert must be a multiple of 64";
    } else if (c.d_ff < 64 || c.d_ff % 64) return "d_ff must be a multiple of 64";
    if (!(c.rope_base > 1.f) || !(c.rms_eps >= 0.f)) return "bad rope_base / rms_eps";
    return nullptr;
}

void plan_model(ModelRT &m, const deer_model_cfg &c, int max_batch, int max_seq) {
    m.c = c;
    m.n_qkv = (c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
    m.kattn = c.n_q_heads * c.head_dim;
    m.F = c.n_experts ? c.d_ff_expert : c.d_ff;
    // a small dense model runs its unsplit residual GEMMs in 32-column workgroups (k_gemm_narrow)
    m.ssq_sub = (!c.n_experts && c.d_model <= NARROW_MAX_D) ? 4 : 1;
    size_t d = c.d_model;
    m.off_embed = 0;
    m.off_lm = align_up((size_t)c.vocab * d * 2);
    m.off_layers = m.off_lm + align_up(d * (size_t)c.vocab * 2);
    m.lo_qkv = 0;
    m.lo_o = m.lo_qkv + align_up(d * m.n_qkv * 2);
    m.lo_router = m.lo_o + align_up((size_t)m.kattn * d * 2);
    m.lo_gu = m.lo_router + (c.n_experts ? align_up(d * CG * 2) : 0);
    m.exp_gu_bytes = align_up(d * 2 * m.F * 2);
    m.exp_d_bytes = align_up((size_t)m.F * d * 2);
    const size_t ne = c.n_experts ? c.n_experts : 1;
    m.lo_d = m.lo_gu + m.exp_gu_bytes * ne;
    m.layer_bytes = m.lo_d + m.exp_d_bytes * ne;
    m.weight_bytes = m.off_layers + m.layer_bytes * c.n_layers;
    m.kv_head_stride = (size_t)max_seq * c.head_dim;
    m.kv_seq_stride = m.kv_head_stride * c.n_kv_heads;
    m.kv_layer_stride = m.kv_seq_stride * max_batch;
    m.kv_k_base = 0;
    m.kv_v_base = m.kv_layer_stride * c.n_layers;
    m.kv_bytes = align_up(2 * m.kv_layer_stride * c.n_layers * 2);
}

// The drafter's prefill has buffers of its own, for passes of up to BESIDE_TILES row tiles.  Larger ones fill the chip by
// themselves (105 row tiles of the 4B pair 16.28 ms one after the other, 16.08 beside each other; 128 of the 8B pair 105.0 and
// 105.4); a drafter of fewer than BESIDE_LAYERS layers does not repay the fork and the join (the tiny pair's request: 8 us
// longer); two mixtures share the routing buffers.
constexpr int BESIDE_TILES = 64, BESIDE_LAYERS = 4;
constexpr size_t BESIDE_PART_FLOATS = 16 << 20;   // split-K partials, at most
bool beside_ok(const deer_init_params &p) { return p.drafter.n_layers >= BESIDE_LAYERS && !(p.target.n_experts && p.drafter.n_experts); }

// Carves the workspace; with base == nullptr only computes the size.
void plan_work(Work &w, const deer_init_params &p, char *base) {
    const int B = p.max_batch;
    const int MAXT = std::max(2 * B, PREFILL_TILES), MAXR = MAXT * 32;
    const int PARTR = std::max(2 * B, PART_TILES_MIN) * 32;
    const deer_model_cfg &t = p.target, &d = p.drafter;
    const size_t dmax = std::max(t.d_model, d.d_model);
    const size_t kattn = std::max(t.n_q_heads * t.head_dim, d.n_q_heads * d.head_dim);
    const size_t fmax = std::max(t.n_experts ? t.d_ff_expert : t.d_ff, d.n_experts ? d.d_ff_expert : d.d_ff);
    const size_t kb = std::max(kattn, fmax);
    const size_t hq = std::max(t.n_q_heads, d.n_q_heads);
    const size_t hdmax = std::max(t.head_dim, d.head_dim);
    const size_t V = std::max(t.vocab, d.vocab);
    const size_t lmrows = (size_t)B * 32;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return base ? base + o : nullptr; };
    // what the host uploads when sequences enter lies together, for one copy: the state, the tile descriptors of the first
    // prefill pass of each model, the prompts
    w.up = take(0);
    w.st.len = (int *)take(B * 4); w.st.dr_len = (int *)take(B * 4); w.st.pending = (int *)take(B * 4);
    w.st.ing_n = (int *)take(B * 4); w.st.finished = (int *)take(B * 4);
    w.up_desc = off;
    w.pf_desc[0] = (int4 *)take((size_t)MAXT * sizeof(int4)); w.pf_desc[1] = (int4 *)take((size_t)MAXT * sizeof(int4));
    w.up_ids = off;
    w.ids = (int *)take((size_t)B * p.max_seq * 4);
    w.st.ing_tok = (int *)take((size_t)B * 32 * 4);
    w.rm.pos = (int *)take(MAXR * 4); w.rm.limit = (int *)take(MAXR * 4);
    w.rm.slot = (int *)take(MAXR * 4); w.rm.seq = (int *)take(MAXR * 4); w.rm.qrow = (int *)take(MAXR * 4); w.rm.grow = (int *)take(MAXR * 4);
    w.rm.tile_seq = (int *)take(MAXT * 4);
    w.cs = (float2 *)take((size_t)MAXR * 64 * sizeof(float2));
    w.theta[0] = (double *)take(64 * 8); w.theta[1] = (double *)take(64 * 8);
    w.h = (float *)take((size_t)MAXR * dmax * 4);
    w.ssq = (float *)take((size_t)MAXR * std::max<size_t>(dmax / CG, std::min<size_t>(dmax, NARROW_MAX_D) / 32) * 4);
    w.xa_hi = (uint4 *)take((size_t)MAXT * (dmax / 16) * 1024); w.xa_lo = (uint4 *)take((size_t)MAXT * (dmax / 16) * 1024);
    w.xb_hi = (uint4 *)take((size_t)MAXT * (kb / 16) * 1024); w.xb_lo = (uint4 *)take((size_t)MAXT * (kb / 16) * 1024);
    w.q_hi = (uint4 *)take((size_t)MAXT * (kattn / 16) * 1024); w.q_lo = (uint4 *)take((size_t)MAXT * (kattn / 16) * 1024);
    w.part = (float *)take((size_t)PARTR * PART_COLS * 4); w.part_floats = (size_t)PARTR * PART_COLS;
    w.opart = (float *)take((size_t)std::max(64, MAXT) * hq * (32 * hdmax + 64) * 4);
    w.logits[0] = (float *)take(lmrows * V * 4); w.logits[1] = (float *)take(lmrows * V * 4);
    w.stat = (RowStat *)take(lmrows * (V / CG) * sizeof(RowStat));
    w.res[0] = (RowResult *)take(lmrows * sizeof(RowResult)); w.res[1] = (RowResult *)take(lmrows * sizeof(RowResult));
    w.ao.accept_len = (int *)take(B * 4); w.ao.n_committed = (int *)take(B * 4); w.ao.committed = (int *)take((size_t)B * 32 * 4);
    w.acc_part = (AccPart *)take((size_t)B * ACC_NB * sizeof(AccPart));
    for (const deer_model_cfg *mc : {&t, &d}) {
        if (!mc->n_experts || w.route_e) continue;
        const size_t tiles = 128 + (size_t)MAXR * 8 / 32, n_items = 128 + (size_t)MAXR * 8 / 64;   // 32-pair tiles and 64-pair items: the last of an expert may be short
        w.route_e = (int *)take((size_t)MAXR * 8 * 4); w.route_w = (float *)take((size_t)MAXR * 8 * 4);
        w.moe_touched = (unsigned long long *)take(8);
        w.pairs = (int *)take((size_t)128 * MAXR * 4);
        w.moe_out = (float *)take((size_t)MAXR * 8 * dmax * 4);
        w.items = (int4 *)take((1 + n_items) * sizeof(int4));
        w.act_hi = (uint4 *)take(tiles * (fmax / 16) * 1024); w.act_lo = (uint4 *)take(tiles * (fmax / 16) * 1024);
        w.xg_hi = (uint4 *)take(tiles * (dmax / 16) * 1024); w.xg_lo = (uint4 *)take(tiles * (dmax / 16) * 1024);
    }
    {
        const size_t ng = (size_t)(std::max(std::max(t.d_model, d.d_model), 4 * (int)fmax) / CG + 64) * MAXT, na = (size_t)MAXT * hq;
        w.cnt_bytes = (2 * (ng + na) + (size_t)B) * 4;
        w.cnt_base = take(w.cnt_bytes);
        int *cnt = (int *)w.cnt_base;
        w.gemm_cnt = cnt; w.attn_cnt = cnt ? cnt + ng : nullptr;
        w.beside.gemm_cnt = cnt ? cnt + ng + na : nullptr; w.beside.attn_cnt = cnt ? cnt + 2 * ng + na : nullptr;
        w.acc_cnt = cnt ? cnt + 2 * (ng + na) : nullptr;
    }
    if (beside_ok(p)) {   // the drafter's own set
        PassBufs &b = w.beside;
        // no more than max_batch sequences of max_seq slots ever need: T row tiles; A attention tiles, of one sequence each;
        // AP partial tiles (a key range holds at least four key tiles); shares of K (eight at most, in blocks of 128 x 256;
        // pieces only beside more than 256 whole blocks, which is above the cap)
        const int key_tiles = p.max_seq / 32, T = (int)std::min<size_t>(BESIDE_TILES, (size_t)B * key_tiles), R = T * 32;
        const size_t A = std::min<size_t>(MAXT, (size_t)B * key_tiles), AP = std::min<size_t>(std::max(64, MAXT), A * ((key_tiles + 3) / 4));
        const size_t F = d.n_experts ? d.d_ff_expert : d.d_ff, wide = std::max<size_t>((size_t)(d.n_q_heads + 2 * d.n_kv_heads) * d.head_dim, std::max<size_t>(2 * F, d.d_model));
        const size_t dd = d.d_model, da = (size_t)d.n_q_heads * d.head_dim, db = std::max(da, F);
        b.rm.pos = (int *)take(R * 4); b.rm.limit = (int *)take(A * 32 * 4); b.rm.slot = (int *)take(R * 4); b.rm.seq = (int *)take(R * 4);
        b.rm.qrow = (int *)take(R * 4); b.rm.grow = (int *)take(A * 32 * 4); b.rm.tile_seq = (int *)take(A * 4);
        b.cs = (float2 *)take((size_t)R * 64 * sizeof(float2));
        b.h = (float *)take((size_t)R * dd * 4);
        b.ssq = (float *)take((size_t)R * (dd / 32) * 4);
        b.xa_hi = (uint4 *)take((size_t)T * (dd / 16) * 1024); b.xa_lo = (uint4 *)take((size_t)T * (dd / 16) * 1024);
        b.xb_hi = (uint4 *)take((size_t)T * (db / 16) * 1024); b.xb_lo = (uint4 *)take((size_t)T * (db / 16) * 1024);
        b.q_hi = (uint4 *)take(A * (da / 16) * 1024); b.q_lo = (uint4 *)take(A * (da / 16) * 1024);
        b.part_floats = std::min<size_t>(BESIDE_PART_FLOATS, (size_t)8 * ((T + BK_RT - 1) / BK_RT * BK_RT * 32) * ((wide + 255) / 256 * 256));
        b.part = (float *)take(b.part_floats * 4);
        b.opart = (float *)take(AP * d.n_q_heads * (32 * d.head_dim + 64) * 4);
    }
    w.stamps = (unsigned long long *)take((size_t)STAMP_MAX_BLOCKS * 8 * 8);
    w.bytes = off;
}

const char *check_params(const deer_init_params *p) {
    if (!p) return "null params";
    if (p->max_batch < 1 || p->max_batch > 1024) return "max_batch out of range";
    if (p->max_k < 1 || p->max_k > 32) return "max_k must be in 1..32";
    if (p->max_seq < 64 || p->max_seq % 64) return "max_seq must be a positive multiple of 64";
    if (const char *e = check_model(p->target)) return e;
    if (const char *e = check_model(p->drafter)) return e;
    if (p->target.vocab != p->drafter.vocab) return "target and drafter must share the vocabulary";
    if (p->mask_token_id < 0 || p->mask_token_id >= p->drafter.vocab) return "mask_token_id outside the vocabulary";
    if (p->eos_token_id >= p->target.vocab) return "eos_token_id outside the vocabulary";
    return nullptr;
}

// ---------------------------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------------------------
// Rounds of streaming workgroups.  With several row-tile groups those of one (column group, K split) pair share an XCD (see
// k_gemm_rows), so it is an XCD's 32 compute units that must hold them: 20 column groups in 12 row-tile groups are 240
// workgroups, but three column groups on some XCDs, 36 workgroups each (4B down, 24 row tiles: 155 us, at 20 row tiles 86).
int stream_rounds(int N, int S, int zg) {
    const int pairs = N / CG * S;
    return zg > 1 ? ((pairs + 7) / 8 * zg + 31) / 32 : (pairs + 255) / 256;
}
// K splits per column group: as many as keep the launch within one wave of workgroups (rounded down: a second
// wave of workgroups costs more than idle CUs).  Measured on MI355X with the 8B- and 4B-shaped matrices: the split-K
// tail (partial store, arrival, the last workgroup's sum) makes ~224 workgroups the best target for matrices with up
// to 256 k-steps, 256 for longer contractions; at most 8 splits; none for contractions of up to 64 k-steps.
int choose_split(int N, int KS, int zgroups) {
    const int blocks = (N / CG) * zgroups;
    const int target = KS > 256 ? 256 : 224;
    int S = std::max(1, target / blocks);
    // the workgroup that finishes a column group sums S partial tiles (about 0.25 us each) before its epilogue:
    // beyond 8 splits that costs more than the shorter streams save (drafter down projection, 7 column groups:
    // 19 splits 22.8 us, 8 splits 18.5 us)
    S = std::min(S, 8);
    // a short contraction (the drafter's d = 896: 56 k-steps) is not split at all: the partial store, the arrival
    // and the last workgroup's sum cost more than streaming a 128-column slab from one workgroup (2.44 -> 2.36 ms per draft pass)
    if (KS <= 64) S = 1;
    S = std::min(S, std::max(1, KS / 16));           // at least 16 k-steps per workgroup
    S = std::min<int>(S, (int)(PART_COLS / (size_t)N));
    S = std::max(S, 1);
    // Fewer where that saves a round on some XCDs and leaves a wave a chain of up to eight k-steps (drafter down, 5 and 6 row tiles,
    // 7 and 6 shares: 16.7 and 17.4 us, in 6 and 5 shares 12.8 and 13.4).  Not with longer chains, whose sums are further off (error against
    // 64 bits, drafter down at 7, 9 and 11 row tiles in 5, 4 and 3 shares 0.97, 1.00 and 1.03e-7, in one fewer 0.99, 1.04 and 1.15e-7;
    // 1536 x 8960 at 3 in 7 shares 1.05, in 6 1.07e-7).  And not where it saves none: the router, one column group, has at most
    // eight pairs, one to an XCD, however many shares, and its shares are what spreads it over the XCDs (128 x 2048 over 33, 66 and
    // 128 row tiles in 6, 6 and 3 shares: 19, 35 and 51 us, in one 33, 53 and 60).
    for (int s = S - 1; s >= 1 && KS <= 64 * s; --s)
        if (stream_rounds(N, s, zgroups) < stream_rounds(N, S, zgroups)) S = s;
    return S;
}

// deer_debug_gemm_stamps: the chosen launch and the one after it record their workgroups' stamps, each in its half of
// the buffer (zeroed at the start of the pass); null for every other launch or one with too many workgroups.
unsigned long long *stamp_buffer(deer_ctx *c, size_t workgroups) {
    const int stamp_rel = c->gemm_launch_idx - c->stamp_launch;
    if (c->stamp_launch < 0 || c->cur_pass_model != c->stamp_model || (stamp_rel != 0 && stamp_rel != 1) ||
        workgroups > (size_t)STAMP_MAX_BLOCKS / 2)
        return nullptr;
    c->stamp_blocks = STAMP_MAX_BLOCKS;
    return c->wk.stamps + (size_t)stamp_rel * (STAMP_MAX_BLOCKS / 2) * 8;
}

// What a GEMM launch takes, in microseconds: rounds of workgroups on 256 compute units, a fixed part for the first loads
// and the epilogue, a part per k-step of a workgroup, and what the shares of a split K cost.  The constants are fitted to
// launches of the 4B, 8B and drafter matrices (K = 896 .. 12288, N = 896 .. 24576) over 2 .. 128 row tiles and are good to
// about 15 %; the choice between kernels needs no more, since near a boundary both take the same time.
// Streaming kernel with MT row tiles per workgroup, microseconds per k-step of a workgroup: pairs 0.125 (8B gate/up at 16 row
// tiles: 6 rounds, 227 us; O at 10 and 12 42, measured 41), in one round of 300 or more 0.134 (8B down at 14 and 16 108 and 113;
// 4B down at 10 and 12, two shares, 52 and 53); one tile 0.075 (8B down at 5 row tiles 72, 4B down at 9 57, mixture's QKV at 12
// 36), of short contractions 0.07 (6144 x 1024 over 6 to 8 17, 2560 x 1536 over 11 23), of an odd number of many tiles, whose
// weights come from L2 once per tile, 0.1.  Where more rounds on some XCDs than over the whole chip are needed, each of these costs its k-steps,
// but not the fixed part; with shares it begins while others meet (4B down at 24 row tiles 152 us, O at 11 45, drafter down at
// 7, 9, 11 and, in pairs, 18 and 24: 18.5, 20.4, 24.0, 32.8 and 40.6).
double stream_us(int N, int KS, int MT, int zg, int S) {
    const int rounds = stream_rounds(N, S, zg), even = (N / CG * S * zg + 255) / 256;   // even: if the XCDs shared the workgroups evenly
    const double per = (double)KS / S, loop = per * (MT == 2 ? (rounds == 1 && per >= 300 ? 0.134 : 0.125) : zg > 16 ? 0.1 : KS >= BK_SHORT ? 0.075 : 0.07);
    return 5.0 + even * (MT == 2 ? 5.0 : 4.0) + rounds * loop + (S > 1 ? 6.0 - (rounds - even) * (MT == 2 ? 2.0 : 4.0) : 0.0);
}
// Narrow workgroups of a small model: rounds of them (ids are padded to 8 column groups, see k_gemm_narrow) on 256 compute
// units.  Fitted to O projections of N = 256 .. 1024, K = 256 .. 1024 and QKV of N = 512 .. 3072 over 1 .. 105 row tiles;
// d = 896: O 5.1 us at 1 tile, 9.3 at 16, 17 at 31, 67 at 105, QKV 7.3, 11.4, 18.4 and 58; d = 256: O 4.1, 4.5, 6.1 and 12.4;
// d = 1024 with 16 kv heads: QKV 7.4, 18, 40 and 127.
double narrow_us(int N, int KS, int ntiles, bool qkv) {
    const double r = (N / (qkv ? 64 : 32) + 7) / 8 * 8 * ntiles / 256.0;
    return qkv ? 5.6 + 0.04 * KS + (3.2 + 0.05 * KS) * std::max(0.0, r - 1.0) : 4.0 + 0.035 * KS + (1.6 + 0.067 * KS) * std::max(0.0, r - 1.5);
}
// Passes of up to SLIM_TILES row tiles, one round of workgroups: a fixed part and behind it the larger of HBM's time for the
// weights (6.5 TB/s) and a compute unit's for what its workgroups draw (62 KB per microsecond).  Fitted to launches of the
// 4B, 8B, 30B-A3B and drafter matrices over one and two row tiles (see k_gemm_slim; microseconds measured / estimated, 8B O
// in 224 wide workgroups 13.2 / 13.4, in 256 slim ones 11.0 / 11.6, drafter down 11.7 / 11.9 and 7.4 / 7.8).
int share_steps(int KS, int S) { return (KS + 8 * S - 1) / (8 * S) * 8; }   // k-steps of a share: whole rounds of the eight waves
double small_us(double base, int N, int KS, int wgs, int S, int frags) {   // frags: 1 KB fragments per k-step of a workgroup
    const double hbm = (double)N * KS * 32.0 / 6.5e6, cu = std::ceil(wgs / 256.0) * std::min(KS, share_steps(KS, S)) * frags / 62.0;
    return base + std::max(hbm, cu);
}
double stream_small_us(int N, int KS, int MT, int zg, int S) {
    return small_us(MT == 2 ? (S > 1 ? 14.0 : 12.0) : (S > 1 ? 8.2 : 5.6), N, KS, N / CG * S * zg, S, 4 + 2 * MT);
}
// The streaming kernel against the blocked one: of few row tiles the lower of its two estimates, since the blocked kernel's own
// is too low there (four row tiles of gate/up, microseconds streaming / blocked and their estimates: 9728 x 896 18.1 / 19.1,
// 16.4 or 20.8 / 19.7; 11264 x 1408 23.6 / 29.8, 22.6 or 25.3 / 23.6; 11776 x 2944 32.3 / 46.5, 35.7 or 33.0 / 34.2).
double stream_or_small_us(int N, int KS, int MT, int zg, int S) {
    const double us = stream_us(N, KS, MT, zg, S);
    return MT * zg <= SLIM_TILES ? std::min(us, stream_small_us(N, KS, MT, zg, S)) : us;
}
// k_gemm_slim for one GEMM of a pass; C == 0: the wide kernels
struct SlimPlan { int C = 0, S = 1, ngrp = 0, pairs = 0; double us = 1e30; };
SlimPlan plan_slim(int epi, int N, int KS, int ntiles, int hd, int ssq_sub, size_t part_floats) {
    SlimPlan best;
    // a residual GEMM leaves one sum of squares per row and workgroup: its width is what the pass keeps
    const int C = epi == EPI_RESID ? 4 / ssq_sub : 2, ngrp = N / (32 * C);
    if (ntiles > SLIM_TILES || C > 2 || (epi != EPI_RESID && epi != EPI_QKV && epi != EPI_SWIGLU)) return best;
    // one workgroup per compute unit, padding of the ids included (a second one on some would take as long again); at most
    // eight shares (they are loaded together)
    for (int S = 1; S <= 8 && (ngrp * S + 7) / 8 * 8 * ntiles <= 256; ++S) {
        if (S > 1 && (KS < 16 * S || (size_t)ngrp * S * ntiles * 1024 * C > part_floats)) break;
        if ((S - 1) * share_steps(KS, S) >= KS) continue;   // (72 k-steps: 4 shares would be 24, 24, 24 and none)
        const double us = small_us((S > 1 ? 6.0 : 4.7) + 0.4 * (C - 1), N, KS, ngrp * S * ntiles, S, C + 2);
        if (us < best.us) best = SlimPlan{C, S, ngrp, epi == EPI_SWIGLU || (epi == EPI_QKV && hd == 128), us};
    }
    // Where it is the stream that counts, it runs at 6.0 TB/s: the workgroups draw the activations twice as often as wide ones
    // (18944 x 3584 over one row tile 31.9 wide and 33.3 slim; 12288 x 4096 24.5 and 23.5).
    best.us = std::max(best.us, (best.S > 1 ? 6.0 : 4.7) + 0.4 * (C - 1) + (double)N * KS * 32.0 / 6.0e6);
    return best;
}
// shares that meet through memory (megabytes): cheap while the L2s hold them
double meet_us(double mb) { return mb <= 20.0 ? 0.2 * mb : 4.0 + 0.55 * (mb - 20.0); }
// Blocked kernel: NB = 4 (128 x 256 per workgroup: 0.3 to 0.4 us per k-step, the more the busier the chip) or NB = 2
// (128 x 128: 0.16 us with 64 workgroups, 0.24 with one per compute unit, 0.225 to 0.235 with more).
struct BlockPlan { int NB = 2, S = 1; bool deep = false; double us = 1e30; int full = 0, G = 0, piece = 0; };   // full: blocks run whole, 0: all (see BlockDeal)
BlockPlan plan_block(int N, int KS, int ntiles, bool lm_head, bool mixture, size_t part_floats) {
    BlockPlan best;
    const int nrb = (ntiles + BK_RT - 1) / BK_RT;
    // 128 columns per wave keep K in one chain of sums (see BK_SHORT): only in large launches (1024 rows on, 128 blocks of
    // 256 x 256), where it is the chip's rate that counts and no kernel before this one cut the chain either; not beside a
    // mixture, where a rounding can send a row to another expert.  (LM heads of fewer rows would gain by it - 16 row
    // tiles, 151936 columns, mean of d = 4096 and 896: 793 against 865 us, 2 to 3 % of an iteration of 16 sequences - but
    // their logits' own error is 2 to 2.8 times the streaming kernel's then.)
    const bool wide_ok = !mixture && ntiles >= 32 && ((ntiles + 7) / 8) * ((N / CG + 1) / 2) >= 128;
    for (int NB = wide_ok ? 4 : 2; NB >= 2; NB -= 2) {
        const int ncb = (N + 64 * NB - 1) / (64 * NB);
        for (int S = 1; S <= (lm_head ? 1 : 8); ++S) {
            const int per = (KS + S - 1) / S;
            if (S > 1 && (per < 16 || (S - 1) * per >= KS)) continue;                          // every share has k-steps
            const double tile_bytes = 4.0 * S * nrb * ncb * 128 * 64 * NB;
            if (S > 1 && tile_bytes > 4.0 * (double)part_floats) continue;
            // rounds of workgroups: two share a compute unit and fill each other's gaps
            const double q = (double)nrb * ncb * S / 256.0;
            const double units = q <= 1.0 ? 1.0 : q > 2.0 ? 0.5 * (q + std::ceil(q)) : NB == 4 ? 2.0 : 1.45 + 0.5 * (q - 1.0);
            // fewer workgroups get more of the L2s each
            const double step = NB == 4 ? (q <= 1.0 ? 0.30 + 0.09 * q : q <= 2.0 ? 0.36 : 0.40) : (q <= 1.0 ? 0.15 + 0.09 * q : q <= 2.0 ? 0.225 : 0.235);
            const double us = 10.0 + units * per * step + (S > 1 ? S + meet_us(tile_bytes * 1e-6) : 0.0);
            // (short contractions: the ring of 8 takes 2 us more; of 128 k-steps, rings of 4 / 8: 12288 columns over 3, 6 and 8 row tiles
            // 28.6 / 26.4, 40.1 / 38.6, 40.8 / 39.0, 4096 over 18, 20 and 28 42.0 / 40.8, 42.2 / 41.1, 45.4 / 43.5, 5120 over 7 and 18 27.5 / 29.0, 44.6 / 42.7)
            if (us < best.us) best = BlockPlan{NB, S, NB == 2 && q <= 1.0 && KS >= BK_SHORT, us};
        }
        // More blocks than compute units: an equal number of whole blocks for each, the rest in pieces of at least an eighth
        // of a block.  A compute unit's rate hardly depends on how many workgroups share it, so that a launch takes the k-steps
        // of the fullest one.  Microseconds, last blocks whole / in pieces: 4B at 105 row tiles O 158 / 132, down 330 / 288 (both
        // against the best uniform shares); 8B gate/up at 9 tiles 170 / 142; half of the last round full: 8B gate/up at 7 and 8
        // tiles 112 / 103 and 116 / 105, QKV at 32 121 / 107, mixture's QKV at 64 106 / 96, O at 96 110 / 103, but the 4B's QKV
        // at 105 tiles, in blocks of 128 x 256, 198 / 206; LM heads 591 / 580 (d = 4096, 7 tiles), 182 / 190 (2048, 4 tiles).
        const int blocks = nrb * ncb, full = blocks / 256 * 256, rest = blocks - full;
        if (full > 0 && rest > 0 && KS >= 32) {
            int G = std::min(256, rest * 8);
            const int piece = std::max(16, (rest * KS + G - 1) / G);
            G = ((rest * KS + piece - 1) / piece + 7) / 8 * 8;
            const double us = 10.0 + ((double)full / 256.0 * KS + piece) * (NB == 4 ? 0.40 : 0.235) + meet_us((G + rest) * 128.0 * 64 * NB * 4e-6);
            if (2.0 * G * 128 * 64 * NB <= (double)part_floats && us < best.us) best = BlockPlan{NB, 1, false, us, full, G, piece};
        }
    }
    return best;
}

// deer_debug_gemm_block: the given form, with as many of the K shares as have k-steps and fit the partials' buffer
BlockPlan forced_block(const deer_ctx *c, int N, int KS, int ntiles, bool lm_head) {
    BlockPlan bp{c->force_nb, lm_head ? 1 : c->force_S, c->force_nb == 2 && c->force_ring == 8 && KS >= BK_SHORT, 0.0};
    const size_t tile_floats = (size_t)((ntiles + BK_RT - 1) / BK_RT) * ((N + 64 * bp.NB - 1) / (64 * bp.NB)) * 128 * 64 * bp.NB;
    while (bp.S > 1 && ((bp.S - 1) * ((KS + bp.S - 1) / bp.S) >= KS || bp.S * tile_floats > c->wk.part_floats)) --bp.S;
    return bp;
}

template <int EPI>
int launch_gemm(deer_ctx *c, GemmArgs &a, int K, int ntiles, int force_S) {
    a.KS = K / 16;
    // Row tiles go through a workgroup in pairs (the weights are read once per pair) unless the matrix is small:
    // then every tile gets workgroups of its own, which find the weights in their XCD's L2, and the workgroup that
    // finishes a column group runs one epilogue instead of two in a row.  Measured on MI355X: the 0.5B drafter's
    // pass over two row tiles 2.26 -> 1.71 ms, over 16 tiles (batch 8) 3.73 -> 3.39 ms, over 32 tiles 5.56 -> 5.80 ms
    // (pairs stay); of the 8B shape's matrices the 33.6 MB output projection gains up to 8 tiles and the 50.3 MB QKV
    // projection up to 4 (batch 2 verify 5.99 -> 5.82 ms), gate/up and down lose at any tile count.
    constexpr double mt1_bytes = 5.1e7, mt1_product = 2.8e8;
    constexpr int mt1_tiles = 16;
    // (matrix bytes x tiles is capped too: the output projection loses at 16 tiles)
    const double w_bytes = (double)a.N * K * 2.0;
    const bool pairs = ntiles % 2 == 0 && !(ntiles <= mt1_tiles && w_bytes <= mt1_bytes && w_bytes * ntiles <= mt1_product);
    const int MT = pairs ? 2 : 1;
    const int zg = ntiles / MT;
    a.rows_total = ntiles * 32;
    const bool narrow = (EPI == EPI_RESID || (EPI == EPI_QKV && a.hd <= 64 && 64 % a.hd == 0 && a.N % 64 == 0)) && a.ssq_sub == 4 && MT == 1 &&
                        force_S <= 0 && a.KS <= 64;
    const int wide_S = force_S > 0 ? force_S : choose_split(a.N, a.KS, zg);
    SlimPlan sp;
    if (!narrow && force_S <= 0 && a.slim) sp = plan_slim(EPI, a.N, a.KS, ntiles, a.hd, a.ssq_sub, c->wk.part_floats);
    const bool slim = sp.C > 0 && sp.us < 0.98 * stream_small_us(a.N, a.KS, MT, zg, wide_S);
    if constexpr (EPI == EPI_SWIGLU) if (c->slim && pairs && ntiles == 2 && a.KS >= BK_SHORT && wide_S <= 2 && !c->force_nb) {
        // Two row tiles of a matrix too large for a tile per workgroup, of which the streaming kernel has no more than two shares
        // (more fill the chip: three of 8320 and 9216 x 4096 27.4 and 28.6 us, here 27.8 and 29.4; four of 8192 x 5120 27.6 / 29.6,
        // small workgroups of 8192 x 4096 25.8 / 28.0).  Shares of K for one workgroup on every compute unit, for two where one
        // would have the whole of K (microseconds, k_gemm / here: 10240 and 12288 x 4096 34.0 / 29.7 and 35.4 / 31.3, 10240 x
        // 2560 26.0 / 23.4, 12800 x 5120 41.0 / 35.5, 19456 x 2560 in 3 shares 32.2 / 29.3, 24576 x 4096 in 2 51.5 / 49.1, 37888
        // x 3584 in 1 78 / 67 to 75, in 3 62)
        const int ncb = (a.N + 255) / 256, nq = a.KS / SK;
        int S = std::max(1, ncb <= 128 ? 256 / ncb : 512 / ncb);
        S = std::min({S, 8, nq / 4});
        while (S > 1 && ((S - 1) * ((nq + S - 1) / S) >= nq || (size_t)S * ncb * GU_PART > c->wk.part_floats)) --S;
        a.S = S; a.part = c->wk.part; a.counters = c->wk.gemm_cnt;
        a.stamps = stamp_buffer(c, (size_t)ncb * S);
        c->gemm_launch_idx++;
        ProfScope ps(c, 0, (double)a.N * K * 2.0);
        hipLaunchKernelGGL(k_gemm_gateup, dim3((unsigned)(ncb * S)), dim3(256), 0, c->stream, a, ncb, (nq + S - 1) / S);
        LAUNCHCHK(c, "k_gemm_gateup");
        return DEER_OK;
    }
    // Up to 32768 columns the streaming kernel's workgroups of 128 columns go in one round, K shared among their waves, and half
    // as many of 256 with the whole of K in each wave take longer (microseconds streaming / k_lm_head, one row tile: 1024 columns of d = 896 11
    // / 16, of 4096 31 / 47; 32000 of 896 15 / 22, of 4096 46 / 59; two row tiles of 4096 56 / 71; 50304 of 896 26 / 23, of 4096 85 / 66).
    if constexpr (EPI == EPI_LMHEAD) if (c->slim && ntiles <= LM_TILES && a.N > LM_COLS && !c->force_nb) {
        a.stamps = stamp_buffer(c, (size_t)(a.N + 255) / 256);
        c->gemm_launch_idx++;
        ProfScope ps(c, 0, (double)a.N * K * 2.0);
        auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((a.N + 255) / 256), dim3(256), 0, c->stream, a, ntiles); };
        const bool sh = a.KS < BK_SHORT;
        if (ntiles == 1) { if (sh) launch(k_lm_head<4, 1, 2, true, 3>); else launch(k_lm_head<4, 1, 2, false, 3>); }
        else if (sh) launch(k_lm_head<4, 2, 2, true, 2>);
        else launch(k_lm_head<4, 2, 2, false, 2>);
        LAUNCHCHK(c, "k_lm_head");
        return DEER_OK;
    }
    if constexpr (EPI != EPI_ROUTER) if (c->block_gemm > 0 && ntiles > 1) {
        const BlockPlan bp = c->force_nb ? forced_block(c, a.N, a.KS, ntiles, EPI == EPI_LMHEAD)
                                         : plan_block(a.N, a.KS, ntiles, EPI == EPI_LMHEAD, c->p.target.n_experts || c->p.drafter.n_experts, c->wk.part_floats);
        const double old_us = narrow ? narrow_us(a.N, a.KS, ntiles, EPI == EPI_QKV) : slim ? sp.us : stream_or_small_us(a.N, a.KS, MT, zg, wide_S);
        const bool forced = c->force_nb || (c->block_gemm > 0 && c->block_gemm < 128 && ntiles >= 8);   // tests cover it at small sizes
        // Not where the streaming kernel has three or more shares of up to 104 k-steps: its waves' chains of sums, of up to 13, are
        // then shorter than the blocked kernel's (error against 64 bits, 896 x 4864 at 18 and 24 row tiles 0.99 and 1.04e-7, blocked
        // 1.10 and 1.07e-7; chains of 23, 1536 x 8960 at 14, 1.26 and 1.13e-7).  It costs 4 and 9 us there.
        const bool short_chains = !narrow && !slim && wide_S >= 3 && a.KS <= wide_S * BK_SHORT;
        if (forced || (!short_chains && bp.us < 0.97 * old_us)) {
            a.S = bp.S; a.part = c->wk.part; a.counters = c->wk.gemm_cnt;
            const int nrb = (ntiles + BK_RT - 1) / BK_RT, ncb = (a.N + 64 * bp.NB - 1) / (64 * bp.NB), band = block_band(nrb);
            const int blocks = nrb * ncb * a.S;
            const BlockDeal deal{blocks, bp.full ? bp.full : blocks, bp.G, bp.piece, (a.KS + a.S - 1) / a.S};
            const dim3 g((unsigned)block_grid(deal));
            ProfScope ps(c, 0, (double)a.N * K * 2.0);
            auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, g, dim3(256), 0, c->stream, a, ncb, ntiles, band, deal); };
            const bool sh = a.KS < BK_SHORT;
            if (bp.G) {
                if (bp.NB == 4) launch(k_gemm_block<4, 4, EPI, false, true>);
                else if (sh) launch(k_gemm_block<2, 4, EPI, true, true>);
                else launch(k_gemm_block<2, 4, EPI, false, true>);
            } else if (bp.NB == 4) launch(k_gemm_block<4, 4, EPI, false, false>);
            else if (bp.deep) launch(k_gemm_block<2, 8, EPI, false, false>);
            else if (sh) launch(k_gemm_block<2, 4, EPI, true, false>);
            else launch(k_gemm_block<2, 4, EPI, false, false>);
            LAUNCHCHK(c, "k_gemm_block");
            return DEER_OK;
        }
    }
    if (narrow) {
        // an unsplit GEMM of a small model: one workgroup per row tile and 32-column weight block (residual GEMM) or
        // 64-column pair of blocks (QKV: whole heads)
        a.S = 1; a.part = nullptr; a.counters = nullptr;
        const int ngrp = EPI == EPI_RESID ? a.N / 32 : a.N / 64;
        a.stamps = stamp_buffer(c, (size_t)ngrp * ntiles);
        c->gemm_launch_idx++;
        ProfScope ps(c, 0, (double)a.N * K * 2.0);
        const dim3 g1((unsigned)(((ngrp + 7) / 8) * 8 * ntiles));
        if (EPI == EPI_RESID) hipLaunchKernelGGL((k_gemm_narrow<1, EPI_RESID>), g1, dim3(512), 0, c->stream, a, ngrp, ntiles);
        else hipLaunchKernelGGL((k_gemm_narrow<2, EPI_QKV>), g1, dim3(512), 0, c->stream, a, ngrp, ntiles);
        LAUNCHCHK(c, "k_gemm_narrow");
        return DEER_OK;
    }
    if constexpr (EPI == EPI_RESID || EPI == EPI_QKV || EPI == EPI_SWIGLU)
        if (slim) {
            a.S = sp.S; a.part = c->wk.part; a.counters = c->wk.gemm_cnt;
            a.stamps = stamp_buffer(c, (size_t)sp.ngrp * sp.S * ntiles);
            c->gemm_launch_idx++;
            ProfScope ps(c, 0, (double)a.N * K * 2.0);
            const dim3 g1((unsigned)((sp.ngrp * sp.S + 7) / 8 * 8 * ntiles));
            if (sp.C == 2) hipLaunchKernelGGL((k_gemm_slim<2, EPI>), g1, dim3(512), 0, c->stream, a, sp.ngrp, ntiles, sp.pairs);
            else if constexpr (EPI == EPI_RESID) hipLaunchKernelGGL((k_gemm_slim<1, EPI>), g1, dim3(512), 0, c->stream, a, sp.ngrp, ntiles, sp.pairs);
            LAUNCHCHK(c, "k_gemm_slim");
            return DEER_OK;
        }
    a.S = wide_S;
    while (a.S > 1 && (size_t)a.S * a.rows_total * a.N > c->wk.part_floats) --a.S;   // partials must fit their buffer
    a.part = (EPI == EPI_LMHEAD) ? nullptr : c->wk.part;
    a.counters = c->wk.gemm_cnt;
    a.stamps = stamp_buffer(c, (size_t)(a.N / CG) * a.S * zg);
    c->gemm_launch_idx++;
    dim3 grid(a.N / CG, a.S, zg);
    ProfScope ps(c, 0, (double)a.N * K * 2.0);
    if (zg > 1) {   // the row-tile groups of a (column group, K split) pair share an XCD's L2
        const int ncg = a.N / CG, pairs8 = (ncg * a.S + 7) / 8;
        dim3 g1((unsigned)(pairs8 * 8 * zg));
        if (MT == 2) hipLaunchKernelGGL((k_gemm_rows<2, EPI>), g1, dim3(512), 0, c->stream, a, ncg, zg);
        else hipLaunchKernelGGL((k_gemm_rows<1, EPI>), g1, dim3(512), 0, c->stream, a, ncg, zg);
    } else if (MT == 2) hipLaunchKernelGGL((k_gemm<2, EPI>), grid, dim3(512), 0, c->stream, a);
    else hipLaunchKernelGGL((k_gemm<1, EPI>), grid, dim3(512), 0, c->stream, a);
    LAUNCHCHK(c, "k_gemm");
    return DEER_OK;
}

// draw: the pass samples its rows' tokens (Gumbel-max over the perturbed logits): the drafter's pass at T > 0; the target's
// rows only need the maximum and the sum of exponentials
struct LmPlan { bool on; int n_lm, k; float T; uint64_t seed; int k_lo = 0; bool draw = false; int *draft = nullptr; };   // n_lm rows with logits, k per sequence

template <int HD>
int launch_attn(deer_ctx *c, ModelRT &m, int layer, int ntiles, int NS, int NS_head, float scale_log2e, double kv_bytes,
                const NextWeights &nx) {
    Work &w = c->wk;
    const deer_model_cfg &mc = m.c;
    const uint16_t *K = m.kv + m.kv_k_base + (size_t)layer * m.kv_layer_stride;
    const uint16_t *Vt = m.kv + m.kv_v_base + (size_t)layer * m.kv_layer_stride;
    ProfScope ps(c, 1, kv_bytes);
    if (NS_head > 0) {   // few tiles: one workgroup per (tile, query head, key range), merged by the last to arrive
        hipLaunchKernelGGL(k_attn_head<HD>, dim3(mc.n_q_heads * NS_head, ntiles), dim3(512), 0, c->stream, w.q_hi, w.q_lo, K, Vt,
                           m.kv_seq_stride, m.kv_head_stride, w.rm.tile_seq, w.rm.limit, w.rm.grow, w.opart, w.attn_cnt,
                           mc.n_q_heads, mc.n_kv_heads, NS_head, scale_log2e, w.xb_hi, w.xb_lo, nx);
        LAUNCHCHK(c, "k_attn_head");
        return DEER_OK;
    }
    const int HG = (mc.n_q_heads / mc.n_kv_heads + ATT_HEADS - 1) / ATT_HEADS;
    hipLaunchKernelGGL(k_attn<HD>, dim3(mc.n_kv_heads * HG * NS, ntiles), dim3(256), 0, c->stream, w.q_hi, w.q_lo, K, Vt,
                       m.kv_seq_stride, m.kv_head_stride, w.rm.tile_seq, w.rm.limit, w.rm.grow, w.opart,
                       mc.n_q_heads, mc.n_kv_heads, HG, NS, scale_log2e, w.xb_hi, w.xb_lo);
    LAUNCHCHK(c, "k_attn");
    if (NS > 1) {
        const int n_items = ntiles * mc.n_q_heads * (HD / 32) * 2;
        hipLaunchKernelGGL(k_attn_merge<HD>, dim3((n_items + 3) / 4), dim3(256), 0, c->stream, w.opart, w.rm.grow, NS, mc.n_q_heads, n_items,
                           scale_log2e, w.xb_hi, w.xb_lo);
        LAUNCHCHK(c, "k_attn_merge");
    }
    return DEER_OK;
}

// Up to how many pairs per expert, on average over all experts, a mixture's projections run in k_gemm_moe; with more of them
// experts of more than 32 pairs, whose weights that kernel reads twice, become frequent.  128 experts of 2048 x 768, top 8,
// microseconds k_gemm_moe / k_moe_block (gate/up: with k_moe_gather; medians of one sweep over three layers, rows spread evenly) at
// 1, 4, 8, 10, 12, 16 row tiles (2 to 32 pairs): gate/up
// 111 / 148, 139 / 169, 149 / 183, 170 / 180, 175 / 184, 230 / 207; down 57 / 65, 69 / 79, 77 / 84, 80 / 82, 86 / 82, 117 / 88.
// 8 experts of 2048 x 5632, top 2, at 1, 2, 4 row tiles (8 to 32): gate/up 69 / 83, 76 / 85, 131 / 88; down 68 / 91, 69 / 92, 129 / 93.
// Small experts keep lower lines, which the tests of what the host launches state (128 experts of 256 x 128 would gain 8 and
// 1 us a launch up to 16 pairs).
constexpr int MOE_GATEUP_PAIRS = 24, MOE_DOWN_PAIRS = 20, MOE_SMALL_GATEUP_PAIRS = 14, MOE_SMALL_DOWN_PAIRS = 12;
constexpr size_t MOE_SMALL_BYTES = 1 << 20;   // of an expert's gate/up matrix

// From how many layers on a pass that only fills the caches leaves out what its last layer would do behind them.  Leaving it out is
// never slower (8 layers of the mixture over 2048 ids 7384 -> 6617 us, 12 of the 4B over 8 prompts 16761 -> 15387, 36 of the 8B over
// 4096 ids 108.3 -> 105.4 ms, 36 of the 4B over 201 ids 7019 -> 6851 us), so the line is no measured one: shorter models run
// whole because most parity tests reach the GEMMs of many row tiles through the prompts of models of one or two layers, and
// would no longer run O, gate/up and down there.  It costs a short drafter, and the tiny pair's request 8 of 40 launches.
constexpr int CACHES_ONLY_LAYERS = 5;

// One forward pass of `model` over the rows described by the row metadata: ntiles tiles of GEMM rows, n_attn attention tiles.
// rows_desc: how the first launch finds the pass's rows.
int run_pass(deer_ctx *c, int model, int ntiles, int n_attn, int max_limit, const LmPlan &lm, double kv_keys_total,
             const PassRows &rows_desc) {
    ModelRT &m = c->m[model];
    Work &w = c->wk;
    const deer_model_cfg &mc = m.c;
    const int d = mc.d_model, hd = mc.head_dim, rows = ntiles * 32, ncg_d = d / CG;
    c->gemm_launch_idx = 0;
    c->cur_pass_model = model;
    // Not for a mixture: with it a row of the full-size mixture's test that lies between two experts went to the other one than
    // in the reference.  (Any order of sums can do that.  A mixture's key ranges per head and its launches in pieces have
    // changed theirs too, without such a row in the tests; what it would gain here has not been set against that.)
    const bool slim = c->slim && !mc.n_experts && ntiles <= SLIM_TILES && d <= SLIM_MAX_D;
    const int ssq_sub = m.ssq_sub == 4 ? 4 : slim ? 2 : 1;   // what the pass's residual GEMMs leave: one sum of squares per 32, 64 or 128 columns
    hipStream_t s = c->stream;
    if (c->stamp_launch >= 0 && model == c->stamp_model) (void)hipMemsetAsync(w.stamps, 0, (size_t)STAMP_MAX_BLOCKS * 64, s);
    prof_close(c);
    hipLaunchKernelGGL(k_pass_begin, dim3(ncg_d + 2, std::max(ntiles, n_attn)), dim3(256), 0, s, rows_desc, w.rm, (const uint16_t *)(m.w + m.off_embed),
                       w.h, w.xa_hi, w.xa_lo, w.ssq, d, ncg_d, ssq_sub, m.theta, w.cs, hd / 2, ntiles, n_attn);
    LAUNCHCHK(c, "k_pass_begin");
    const int nkt = (max_limit + 31) / 32;
    // key-range splits: aim at two workgroups per compute unit; a split holds at least four key tiles; n_attn * NS never
    // exceeds the partial buffer (max(64, most tiles of a pass) tile slots)
    constexpr int ns_target = 256;
    const int attn_items = mc.n_kv_heads * ((mc.n_q_heads / mc.n_kv_heads + ATT_HEADS - 1) / ATT_HEADS) * n_attn;
    int NS = (2 * ns_target + attn_items - 1) / attn_items;
    NS = std::max(1, std::min({NS, MAX_NS, std::max(1, std::max(64, c->max_tiles) / n_attn), (nkt + 3) / 4}));
    // Passes of few tiles (decoding) run attention per query head: (tile, head, key range) workgroups, about one per
    // compute unit, as long as a wave then has at most ATT_HEAD_MAX_TILES key tiles of its range to go through
    int NS_head = 0;
    if (n_attn * mc.n_q_heads <= ns_target) {
        const int ns_max = std::max(1, std::min({ns_target / (n_attn * mc.n_q_heads), ATT_HEAD_MAX_NS, std::max(1, std::max(64, c->max_tiles) / n_attn), (nkt + 7) / 8}));
        // a range's key tiles (0.28 us each with head_dim 128) against the merge, which one compute unit per head runs behind the
        // last of them, about 0.2 us per range (14 heads of 64, 129 key tiles: 17 ranges, one tile per wave, 13.0 us from the
        // launch's first workgroup to its last store, 10 ranges 9.9).  More than ATT_HEAD_NS ranges, which the merge takes in
        // several goes, only where a wave would have too many tiles of fewer (14 heads of 64, one launch: 20000 keys in 16
        // ranges 16.6 us, in 18 17.8; 52000 keys, where 16 do not go, in 18 26.6 and by the kernels for many tiles 42.9; 8 heads
        // of 128: 24000 keys in 16 ranges 25.9, in 29 27.4; 64000 keys in 32 48.6, by the others 68.7)
        auto cost = [&](int n) { return (nkt + n - 1) / n * hd * 0.0022 + (n > 1 ? 1.0 + 0.2 * n : 0.0); };
        for (int n = 1; n <= ns_max; ++n)
            if ((nkt + n - 1) / n <= 8 * ATT_HEAD_MAX_TILES && (NS_head == 0 || (cost(n) < cost(NS_head) && (n <= ATT_HEAD_NS || NS_head > ATT_HEAD_NS)))) NS_head = n;
    }
    const float scale_log2e = (float)(1.4426950408889634 / std::sqrt((double)hd));
    const double kv_bytes = kv_keys_total * mc.n_kv_heads * hd * 2.0 * 2.0;   // K and V rows read per layer
    GemmArgs base{};
    base.ssq_in = w.ssq; base.ncg_in = ncg_d * ssq_sub; base.d_in = d; base.eps = mc.rms_eps;
    base.ssq_sub = ssq_sub; base.slim = slim;
    base.cs = w.cs; base.rm = w.rm; base.qhi = w.q_hi; base.qlo = w.q_lo;
    base.Hq = mc.n_q_heads; base.Hkv = mc.n_kv_heads; base.hd = hd;
    base.h = w.h; base.xhi_out = w.xa_hi; base.xlo_out = w.xa_lo; base.ssq_out = w.ssq;
    base.ahi = w.xb_hi; base.alo = w.xb_lo; base.F = m.F;
    // What the idle workgroups of a split launch pull into their XCD's L2 for the launch after it (passes of one row
    // tile, wide workgroups): the first k-steps of every workgroup of the next GEMM — attention fetches for the output
    // projection, the down projection for the next layer's QKV projection — and, from the QKV projection, the old K,V
    // blocks of the kv head its XCD serves in the per-head attention launch.  Measured (8B target, prefix 4096): verify
    // pass 4.29 -> 4.21 ms; more than 16 KB per 32-column block, or fetching from unsplit launches (after their
    // epilogue) or for gate/up, costs more than it saves.
    // A small dense model (narrow workgroups for its unsplit O and QKV projections, one or two row tiles): attention
    // fetches the output projection's 32-column blocks whole, the split down projection the next layer's QKV blocks.
    const bool small_dense = m.ssq_sub == 4;
    const bool fetch_ahead = ntiles == 1 && !small_dense;
    const bool fetch_ahead_narrow = ntiles <= 2 && small_dense && !mc.n_experts;
    auto next_plan_narrow = [&](const char *W, int N, int K, int NB) {   // NB: 1 residual GEMM, 2 QKV (whole heads)
        NextWeights nx{};
        const int KS = K / 16;
        if (!fetch_ahead_narrow || KS > 64 || N % (32 * NB)) return nx;
        if (NB == 2 && !(hd <= 64 && 64 % hd == 0)) return nx;
        nx.base = W; nx.ncg = N / (32 * NB); nx.nwg = ((nx.ncg + 7) / 8) * 8 * ntiles;
        nx.block_bytes = (long long)KS * 1024; nx.narrow_nb = NB; nx.Z = ntiles;
        return nx;
    };
    auto next_plan = [&](const char *W, int N, int K, int epi) {
        NextWeights nx{};
        if (!fetch_ahead) return nx;
        const int KS = K / 16;
        int S = choose_split(N, KS, 1);
        nx.ncg = N / CG; nx.nblk = 4;
        const SlimPlan sp = slim ? plan_slim(epi, N, KS, 1, hd, ssq_sub, c->wk.part_floats) : SlimPlan{};
        if (sp.C > 0 && sp.us < 0.98 * stream_small_us(N, KS, 1, 1, S)) { S = sp.S; nx.ncg = sp.ngrp; nx.nblk = sp.C; nx.pairs = sp.pairs; }
        else while (S > 1 && (size_t)S * 32 * N > c->wk.part_floats) --S;
        const int per = (KS + S * 8 - 1) / (S * 8);
        nx.base = W; nx.nwg = nx.ncg * S; nx.span = NEXT_SPAN_BYTES;
        nx.block_bytes = (long long)KS * 1024; nx.split_bytes = (long long)8 * per * 1024;
        return nx;
    };
    // Of a pass without logits only the caches are read, so its last layer ends with its K and V rows: no Q columns, no
    // attention, no O, gate/up and down.
    const int n_kv = 2 * mc.n_kv_heads * hd;
    const bool caches_only = !lm.on && mc.n_layers >= CACHES_ONLY_LAYERS && n_kv % CG == 0;
    auto kv_only = [&](int l) { return caches_only && l + 1 == mc.n_layers; };
    // what the QKV launch of layer l multiplies: all of the matrix, or its columns behind Q's
    auto qkv_matrix = [&](int l) { return m.w + m.off_layers + (size_t)l * m.layer_bytes + m.lo_qkv + (kv_only(l) ? (size_t)(m.kattn / 32) * (d / 16) * 1024 : 0); };
    auto qkv_cols = [&](int l) { return kv_only(l) ? n_kv : m.n_qkv; };
    for (int l = 0; l < mc.n_layers; ++l) {
        const char *lw = m.w + m.off_layers + (size_t)l * m.layer_bytes;
        GemmArgs a = base;
        a.W = (const uint4 *)qkv_matrix(l); a.Xhi = w.xa_hi; a.Xlo = w.xa_lo; a.N = qkv_cols(l);
        a.kv = KvView{m.kv + m.kv_k_base + (size_t)l * m.kv_layer_stride, m.kv + m.kv_v_base + (size_t)l * m.kv_layer_stride,
                      m.kv_seq_stride, m.kv_head_stride, c->p.max_seq};
        // whole key tiles that no row of this pass writes (a pass of one tile appends at most 32 rows)
        if (fetch_ahead && NS_head > 0 && c->batch == 1 && 8 % mc.n_kv_heads == 0)
            a.kv_fetch_bytes = std::min(KV_FETCH_MAX_BYTES, std::max(0, (max_limit - 32) / 32) * 32 * hd * 2);
        if (kv_only(l)) { a.Hq = 0; a.kv_fetch_bytes = 0; }
        int rc = launch_gemm<EPI_QKV>(c, a, d, ntiles, 0);
        if (rc) return rc;
        if (kv_only(l)) break;
        const NextWeights nx_o = fetch_ahead_narrow ? next_plan_narrow(lw + m.lo_o, d, m.kattn, 1) : next_plan(lw + m.lo_o, d, m.kattn, EPI_RESID);
        if (hd == 128) rc = launch_attn<128>(c, m, l, n_attn, NS, NS_head, scale_log2e, kv_bytes, nx_o);
        else if (hd == 64) rc = launch_attn<64>(c, m, l, n_attn, NS, NS_head, scale_log2e, kv_bytes, nx_o);
        else rc = launch_attn<32>(c, m, l, n_attn, NS, NS_head, scale_log2e, kv_bytes, nx_o);
        if (rc) return rc;
        a = base;
        a.W = (const uint4 *)(lw + m.lo_o); a.Xhi = w.xb_hi; a.Xlo = w.xb_lo; a.N = d;
        rc = launch_gemm<EPI_RESID>(c, a, m.kattn, ntiles, 0);
        if (rc) return rc;
        if (!mc.n_experts) {
            a = base;
            a.W = (const uint4 *)(lw + m.lo_gu); a.Xhi = w.xa_hi; a.Xlo = w.xa_lo; a.N = 2 * m.F;
            rc = launch_gemm<EPI_SWIGLU>(c, a, d, ntiles, 0);
            if (rc) return rc;
            a = base;
            a.W = (const uint4 *)(lw + m.lo_d); a.Xhi = w.xb_hi; a.Xlo = w.xb_lo; a.N = d;
            if (l + 1 < mc.n_layers)
                a.nx = fetch_ahead_narrow ? next_plan_narrow(qkv_matrix(l + 1), qkv_cols(l + 1), d, 2)
                                          : next_plan(qkv_matrix(l + 1), qkv_cols(l + 1), d, EPI_QKV);
            rc = launch_gemm<EPI_RESID>(c, a, m.F, ntiles, 0);
            if (rc) return rc;
        } else {
            // router -> per-expert grouping -> grouped gate/up and down GEMMs -> ordered combine
            a = base;
            a.W = (const uint4 *)(lw + m.lo_router); a.Xhi = w.xa_hi; a.Xlo = w.xa_lo; a.N = CG;
            a.n_experts = mc.n_experts; a.top_k = mc.top_k; a.route_e = w.route_e; a.route_w = w.route_w;
            a.route_spread = (c->route_spread && (mc.n_experts & (mc.n_experts - 1)) == 0) ? l + 1 : 0;
            rc = launch_gemm<EPI_ROUTER>(c, a, d, ntiles, 0);
            if (rc) return rc;
            const int cap = rows;
            const bool small = m.exp_gu_bytes < MOE_SMALL_BYTES;
            auto few = [&](int pairs) { return rows * mc.top_k < pairs * mc.n_experts; };
            const bool blocked = c->block_gemm > 0 && !few(small ? MOE_SMALL_GATEUP_PAIRS : MOE_GATEUP_PAIRS);
            const bool blocked_down = !few(small ? MOE_SMALL_DOWN_PAIRS : MOE_DOWN_PAIRS);
            // Items of 32 pairs where k_gemm_moe, which multiplies 32 at a time, takes both projections: the row tiles of an expert
            // with more then run beside each other
            const int item_pairs = blocked || blocked_down ? 64 : 32;
            prof_close(c);
            hipLaunchKernelGGL(k_moe_group, dim3(1), dim3(1024), 0, s, w.route_e, w.rm.slot, rows, mc.top_k, cap, item_pairs,
                               w.pairs, w.items, w.moe_touched);
            LAUNCHCHK(c, "k_moe_group");
            MoeArgs ma{};
            ma.cap = cap; ma.pairs = w.pairs; ma.items = w.items;
            ma.ssq_in = w.ssq; ma.ncg_in = ncg_d; ma.d_in = d; ma.eps = mc.rms_eps;
            ma.ahi = w.act_hi; ma.alo = w.act_lo; ma.Fe = m.F; ma.route_w = w.route_w; ma.moe_out = w.moe_out; ma.d = d;
            ma.W = (const uint4 *)(lw + m.lo_gu); ma.wexp_stride = m.exp_gu_bytes / 16; ma.Xhi = w.xa_hi; ma.Xlo = w.xa_lo;
            ma.N = 2 * m.F; ma.KS = d / 16;
            const size_t max_items = (size_t)std::min(mc.n_experts, rows * mc.top_k) + (size_t)rows * mc.top_k / item_pairs;
            auto block_grid_x = [&](int N) { return dim3((unsigned)(8 * ((max_items * ((N + 255) / 256) + 7) / 8))); };
            if (blocked) {
                hipLaunchKernelGGL(k_moe_gather, dim3(ncg_d, (unsigned)max_items), dim3(256), 0, s, w.h, ma, w.xg_hi, w.xg_lo);
                LAUNCHCHK(c, "k_moe_gather");
                ma.Xhi = w.xg_hi; ma.Xlo = w.xg_lo;
            }
            {
                ProfScope ps(c, 0, 0.0);
                auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, block_grid_x(ma.N), dim3(256), 0, s, ma, (ma.N + 255) / 256); };
                // Up to the small experts' line k_gemm_moe sums K in eighths where they are whole stages, as the eight waves of the
                // streaming kernel did that it took over from: a row that lies between two experts then goes where it went.  (Any
                // other order sends one the other way now and then: 8 layers, 128 rows, one of ten sets of weights, and that set's
                // logits 6e-3 off.)
                ma.eighths = few(MOE_SMALL_GATEUP_PAIRS) && ma.KS % (8 * SK) == 0;
                const bool sh = ma.KS < BK_SHORT;
                if (blocked) { if (sh) launch(k_moe_block<MOE_GATEUP, true>); else launch(k_moe_block<MOE_GATEUP, false>); }
                else if (sh && !ma.eighths) launch(k_gemm_moe<MOE_GATEUP, true>);
                else launch(k_gemm_moe<MOE_GATEUP, false>);
            }
            LAUNCHCHK(c, "grouped gate/up");
            ma.W = (const uint4 *)(lw + m.lo_d); ma.wexp_stride = m.exp_d_bytes / 16; ma.Xhi = w.act_hi; ma.Xlo = w.act_lo;
            ma.N = d; ma.KS = m.F / 16; ma.eighths = 0;
            {
                ProfScope ps(c, 0, 0.0);
                auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, block_grid_x(ma.N), dim3(256), 0, s, ma, (ma.N + 255) / 256); };
                if (ma.KS < BK_SHORT) { if (blocked_down) launch(k_moe_block<MOE_DOWN, true>); else launch(k_gemm_moe<MOE_DOWN, true>); }
                else if (blocked_down) launch(k_moe_block<MOE_DOWN, false>); else launch(k_gemm_moe<MOE_DOWN, false>);
            }
            LAUNCHCHK(c, "grouped down");
            prof_close(c);
            hipLaunchKernelGGL(k_moe_combine, dim3(ncg_d, ntiles), dim3(256), 0, s, w.moe_out, w.rm.slot, mc.top_k, w.h, w.xa_hi,
                               w.xa_lo, w.ssq, d);
            LAUNCHCHK(c, "k_moe_combine");
        }
    }
    if (lm.on) {
        const int V = mc.vocab;
        GemmArgs a = base;
        a.W = (const uint4 *)(m.w + m.off_lm); a.Xhi = w.xa_hi; a.Xlo = w.xa_lo; a.N = V;
        a.k = lm.k; a.n_lm = lm.n_lm; a.k_lo = lm.k_lo; a.T = lm.T; a.seed = lm.seed; a.draw = lm.draw ? 1 : 0; a.stat = w.stat; a.ncg_v = V / CG;
        a.logits = (c->p.keep_logits || lm.T > 0.f) ? w.logits[model] : nullptr;
        int rc = launch_gemm<EPI_LMHEAD>(c, a, d, (lm.n_lm + 31) / 32, 1);
        if (rc) return rc;
        prof_close(c);
        hipLaunchKernelGGL(k_rowstat_final, dim3(lm.n_lm), dim3(256), 0, s, w.stat, V / CG, lm.T, w.res[model], lm.k, lm.k_lo, w.st, lm.draft);
        LAUNCHCHK(c, "k_rowstat_final");
    }
    prof_close(c);
    return DEER_OK;
}

// Host image of the block at Work::up: page-locked where it fits (hipMemcpyAsync then needs no copy of its own), valid until
// the stream has been waited for.
char *upload_image(deer_ctx *c, size_t bytes) {
    if (c->h_up && bytes <= c->h_up_bytes) return c->h_up;
    c->h_up_vec.resize(bytes);
    return c->h_up_vec.data();
}
void fill_state(deer_ctx *c, char *img, int B, const int *len, const int *dr_len, const int *pending) {
    const char *up = c->wk.up;
    memcpy(img + ((char *)c->wk.st.len - up), len, (size_t)B * 4);
    memcpy(img + ((char *)c->wk.st.dr_len - up), dr_len, (size_t)B * 4);
    memcpy(img + ((char *)c->wk.st.pending - up), pending, (size_t)B * 4);
    memset(img + ((char *)c->wk.st.ing_n - up), 0, (size_t)B * 4);
    memset(img + ((char *)c->wk.st.finished - up), 0, (size_t)B * 4);
}
struct PrefillPass { std::vector<int4> desc; int n_rows = 0, maxlim = 0; };   // attention tiles (see PassRows), GEMM rows, most visible keys
// The uploads and passes of a prefill; passes[model] and ids must live until the stream has been waited for.
int enqueue_prefill(deer_ctx *c, int batch, const int *ids, const int *lens, const int *pending, size_t total,
                    const std::vector<PrefillPass> (&passes)[2]) {
    Work &w = c->wk;
    // one copy for the state, the first pass's descriptors of each model and the prompts (five copies and a second wait made
    // a short request's prefill 60 us longer)
    const size_t up_bytes = w.up_ids + total * 4;
    char *img = upload_image(c, up_bytes);
    fill_state(c, img, batch, lens, lens, pending);
    for (int model = 0; model < 2; ++model)
        if (!passes[model].empty())
            memcpy(img + ((char *)w.pf_desc[model] - w.up), passes[model][0].desc.data(), passes[model][0].desc.size() * sizeof(int4));
    memcpy(img + w.up_ids, ids, total * 4);
    HIPCHK(c, hipMemcpyAsync(w.up, img, up_bytes, hipMemcpyHostToDevice, c->stream));
    // The two models' caches do not depend on each other.  A prompt's passes leave compute units idle in every launch (its
    // first loads, the meeting of shares, the last round of workgroups), so the drafter's run beside the target's, on a stream
    // of their own with buffers of their own, between two events of the library's stream: 201 tokens through the 4B pair 8.06
    // -> 7.13 ms, 2048 through 8 layers of the mixture with 4 of the drafter 7.60 -> 7.31.  (Not while launches are timed or
    // stamped: those records are of one stream.)
    bool fits = !passes[DEER_TARGET].empty();
    for (const PrefillPass &pa : passes[DEER_DRAFTER]) fits = fits && (pa.n_rows + 31) / 32 <= BESIDE_TILES;
    const bool beside = fits && c->side && !c->prof_on && c->stamp_launch < 0;
    if (beside) HIPCHK(c, hipEventRecord(c->fork, c->stream));
    auto run = [&](int model) -> int {
        for (size_t i = 0; i < passes[model].size(); ++i) {
            const PrefillPass &pa = passes[model][i];
            if (i > 0)
                HIPCHK(c, hipMemcpyAsync(w.pf_desc[model], pa.desc.data(), pa.desc.size() * sizeof(int4), hipMemcpyHostToDevice, c->stream));
            PassRows pr{};
            pr.kind = ROWS_PREFILL; pr.desc = w.pf_desc[model]; pr.ids = w.ids; pr.n_desc = (int)pa.desc.size();
            const LmPlan lm{false, 0, 0, 0.f, 0};
            if (int rc = run_pass(c, model, (pa.n_rows + 31) / 32, pr.n_desc, pa.maxlim, lm, 0.0, pr)) return rc;
        }
        return DEER_OK;
    };
    if (int rc = run(DEER_TARGET)) return rc;
    if (!beside) return run(DEER_DRAFTER);
    HIPCHK(c, hipStreamWaitEvent(c->side, c->fork, 0));
    const hipStream_t own = c->stream;
    c->stream = c->side;
    std::swap((PassBufs &)w, w.beside);
    const int rc = run(DEER_DRAFTER);
    std::swap((PassBufs &)w, w.beside);
    c->stream = own;
    const hipError_t e = hipEventRecord(c->join, c->side), e2 = hipStreamWaitEvent(c->stream, c->join, 0);
    if (rc) return rc;
    if (e != hipSuccess || e2 != hipSuccess) return fail(c, DEER_EHIP, "prefill: %s", hipGetErrorString(e != hipSuccess ? e : e2));
    return DEER_OK;
}
// the host's mirror once the device state is in place
void set_state(deer_ctx *c, int B, const int *len) {
    c->batch = B;
    c->h_len.assign(len, len + B);
    c->h_ing_n.assign(B, 0);
    c->h_finished.assign(B, 0);
    c->state = ST_PREFILLED;
}

}  // namespace

// =============================================================================================
// C ABI
// =============================================================================================
extern "C" {

int deer_query_sizes(const deer_init_params *p, deer_sizes *out) {
    if (!out) return fail(nullptr, DEER_EINVAL, "null output");
    if (p && (p->struct_size != sizeof(deer_init_params) || p->abi_version != DEER_ABI_VERSION))
        return fail(nullptr, DEER_EVERSION, "struct_size/abi_version mismatch");
    if (const char *e = check_params(p)) return fail(nullptr, DEER_EINVAL, "%s", e);
    ModelRT m;
    for (int i = 0; i < 2; ++i) {
        plan_model(m, i == 0 ? p->target : p->drafter, p->max_batch, p->max_seq);
        out->weights[i] = m.weight_bytes;
        out->kv[i] = m.kv_bytes;
    }
    Work w;
    plan_work(w, *p, nullptr);
    out->workspace = w.bytes;
    out->staging = 0;
    return DEER_OK;
}

int deer_init_models(const deer_init_params *p, const deer_buffers *bufs, const deer_sizes *buf_sizes, deer_ctx **out) {
    if (out) *out = nullptr;
    if (!out || !bufs || !buf_sizes) return fail(nullptr, DEER_EINVAL, "null argument");
    deer_sizes need;
    int rc = deer_query_sizes(p, &need);
    if (rc) return rc;
    for (int i = 0; i < 2; ++i) {
        if (!bufs->weights[i] || !bufs->kv[i]) return fail(nullptr, DEER_EINVAL, "null device buffer");
        if (buf_sizes->weights[i] < need.weights[i] || buf_sizes->kv[i] < need.kv[i])
            return fail(nullptr, DEER_ECAPACITY, "weights/kv buffer %d too small", i);
    }
    if (!bufs->workspace) return fail(nullptr, DEER_EINVAL, "null workspace");
    if (buf_sizes->workspace < need.workspace) return fail(nullptr, DEER_ECAPACITY, "workspace too small");
    deer_ctx *c = new (std::nothrow) deer_ctx();
    if (!c) return fail(nullptr, DEER_EINVAL, "out of host memory");
    c->p = *p;
    c->stream = (hipStream_t)p->hip_stream;
    hipError_t e = hipSetDevice(p->device);
    if (e != hipSuccess) { delete c; return fail(nullptr, DEER_EHIP, "hipSetDevice: %s", hipGetErrorString(e)); }
    if (p->device >= 0 && p->device < MAX_DEVICES) {   // this device's address of the static scratch array
        if (!g_scratch_ptr[p->device]) {
            void *ptr = nullptr;
            e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
            if (e != hipSuccess) { delete c; return fail(nullptr, DEER_EHIP, "hipGetSymbolAddress: %s", hipGetErrorString(e)); }
            g_scratch_ptr[p->device] = ptr;
        }
        c->static_scratch = g_scratch_ptr[p->device];
    }
    for (int i = 0; i < 2; ++i) {
        plan_model(c->m[i], i == 0 ? p->target : p->drafter, p->max_batch, p->max_seq);
        c->m[i].w = (char *)bufs->weights[i];
        c->m[i].kv = (uint16_t *)bufs->kv[i];
    }
    plan_work(c->wk, *p, (char *)bufs->workspace);
    c->max_tiles = std::max(2 * p->max_batch, PREFILL_TILES);
    // caches must hold finite values everywhere: masked keys are multiplied by zero weights
    for (int i = 0; i < 2; ++i) {
        e = hipMemsetAsync(bufs->kv[i], 0, need.kv[i], c->stream);
        if (e != hipSuccess) { delete c; return fail(nullptr, DEER_EHIP, "hipMemsetAsync: %s", hipGetErrorString(e)); }
        const deer_model_cfg &mc = c->m[i].c;
        double th[64];
        for (int k = 0; k < mc.head_dim / 2; ++k) th[k] = std::pow((double)mc.rope_base, -2.0 * k / mc.head_dim);
        c->m[i].theta = c->wk.theta[i];
        e = hipMemcpy(c->m[i].theta, th, sizeof(double) * (mc.head_dim / 2), hipMemcpyHostToDevice);
        if (e != hipSuccess) { delete c; return fail(nullptr, DEER_EHIP, "hipMemcpy: %s", hipGetErrorString(e)); }
    }
    if (c->wk.moe_touched) (void)hipMemsetAsync(c->wk.moe_touched, 0, 8, c->stream);
    e = hipMemsetAsync(c->wk.cnt_base, 0, c->wk.cnt_bytes, c->stream);
    if (e != hipSuccess) { delete c; return fail(nullptr, DEER_EHIP, "hipMemsetAsync: %s", hipGetErrorString(e)); }
    e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) { delete c; return fail(nullptr, DEER_EHIP, "hipStreamSynchronize: %s", hipGetErrorString(e)); }
    {   // a few KB of page-locked host memory for the acceptance results (host memory: the device buffers stay the caller's)
        const size_t bytes = (size_t)((const char *)c->wk.ao.committed - (const char *)c->wk.ao.accept_len) + (size_t)p->max_batch * 32 * 4;
        void *hp = nullptr;
        if (hipHostMalloc(&hp, bytes, hipHostMallocDefault) == hipSuccess) {
            void *dp = nullptr;
            c->h_pin = (char *)hp; c->h_pin_bytes = bytes;
            if (hipHostGetDevicePointer(&dp, hp, 0) == hipSuccess) c->h_pin_dev = (char *)dp; else (void)hipGetLastError();
        } else (void)hipGetLastError();
        const size_t up_bytes = std::min<size_t>(c->wk.up_ids + (size_t)p->max_batch * p->max_seq * 4, H_UP_MAX);
        if (hipHostMalloc(&hp, up_bytes, hipHostMallocDefault) == hipSuccess) { c->h_up = (char *)hp; c->h_up_bytes = up_bytes; }
        else (void)hipGetLastError();
    }
    if (c->wk.beside.h) {   // (no stream: the drafter's prefill follows the target's)
        if (hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking) != hipSuccess) c->side = nullptr;
        if (c->side && (hipEventCreateWithFlags(&c->fork, hipEventDisableTiming) != hipSuccess || hipEventCreateWithFlags(&c->join, hipEventDisableTiming) != hipSuccess)) {
            (void)hipStreamDestroy(c->side);
            c->side = nullptr;
        }
        (void)hipGetLastError();
    }
    *out = c;
    return DEER_OK;
}

int deer_load_tensor(deer_ctx *c, int model, int tensor_id, int layer, int expert, const void *src, int src_dtype,
                     int64_t rows, int64_t cols) {
    if (!c) return DEER_EINVAL;
    if (!src || model < 0 || model > 1 || (src_dtype != DEER_F32 && src_dtype != DEER_BF16))
        return fail(c, DEER_EINVAL, "bad model/dtype/pointer");
    ModelRT &m = c->m[model];
    const deer_model_cfg &mc = m.c;
    const int d = mc.d_model, hd = mc.head_dim;
    int64_t er = 0, ec = 0;
    char *dst = nullptr;
    int mode = 0, col_off = 0, K = 0;
    const bool per_layer = tensor_id >= DEER_T_WQ && tensor_id <= DEER_T_ROUTER;
    const bool per_expert = mc.n_experts && (tensor_id == DEER_T_WG || tensor_id == DEER_T_WU || tensor_id == DEER_T_WD);
    if (per_expert && (expert < 0 || expert >= mc.n_experts)) return fail(c, DEER_EINVAL, "expert out of range");
    if (!per_expert && expert >= 0) return fail(c, DEER_EINVAL, "tensor %d takes no expert index", tensor_id);
    const size_t ex = per_expert ? (size_t)expert : 0;
    if (per_layer && (layer < 0 || layer >= mc.n_layers)) return fail(c, DEER_EINVAL, "layer out of range");
    char *lw = m.w + m.off_layers + (size_t)(per_layer ? layer : 0) * m.layer_bytes;
    switch (tensor_id) {
        case DEER_T_EMBED: er = mc.vocab; ec = d; dst = m.w + m.off_embed; break;
        case DEER_T_LM_HEAD: er = d; ec = mc.vocab; dst = m.w + m.off_lm; K = d; break;
        case DEER_T_WQ: er = d; ec = mc.n_q_heads * hd; dst = lw + m.lo_qkv; K = d; break;
        case DEER_T_WK: er = d; ec = mc.n_kv_heads * hd; dst = lw + m.lo_qkv; K = d; col_off = mc.n_q_heads * hd; break;
        case DEER_T_WV: er = d; ec = mc.n_kv_heads * hd; dst = lw + m.lo_qkv; K = d; col_off = (mc.n_q_heads + mc.n_kv_heads) * hd; break;
        case DEER_T_WO: er = m.kattn; ec = d; dst = lw + m.lo_o; K = m.kattn; break;
        case DEER_T_WG: er = d; ec = m.F; dst = lw + m.lo_gu + ex * m.exp_gu_bytes; K = d; mode = 1; break;
        case DEER_T_WU: er = d; ec = m.F; dst = lw + m.lo_gu + ex * m.exp_gu_bytes; K = d; mode = 2; break;
        case DEER_T_WD: er = m.F; ec = d; dst = lw + m.lo_d + ex * m.exp_d_bytes; K = m.F; break;
        case DEER_T_ROUTER:
            if (!mc.n_experts) return fail(c, DEER_EINVAL, "model has no router");
            er = d; ec = mc.n_experts; dst = lw + m.lo_router; K = d; break;
        default: return fail(c, DEER_EINVAL, "unknown tensor id %d", tensor_id);
    }
    if (rows != er || cols != ec) return fail(c, DEER_EINVAL, "tensor %d: expected %lld x %lld, got %lld x %lld", tensor_id,
                                              (long long)er, (long long)ec, (long long)rows, (long long)cols);
    if (tensor_id == DEER_T_EMBED) {
        size_t n = (size_t)rows * cols;
        dim3 grid((unsigned)((n + 255) / 256));
        if (src_dtype == DEER_F32) hipLaunchKernelGGL(k_convert_rows<float>, grid, dim3(256), 0, c->stream, (const float *)src, (uint16_t *)dst, n);
        else hipLaunchKernelGGL(k_convert_rows<uint16_t>, grid, dim3(256), 0, c->stream, (const uint16_t *)src, (uint16_t *)dst, n);
    } else {
        size_t n = (size_t)(K / 8) * cols;
        dim3 grid((unsigned)((n + 255) / 256));
        if (src_dtype == DEER_F32) hipLaunchKernelGGL(k_repack<float>, grid, dim3(256), 0, c->stream, (const float *)src, (uint4 *)dst, K, (int)cols, K / 16, mode, col_off);
        else hipLaunchKernelGGL(k_repack<uint16_t>, grid, dim3(256), 0, c->stream, (const uint16_t *)src, (uint4 *)dst, K, (int)cols, K / 16, mode, col_off);
    }
    LAUNCHCHK(c, "k_repack");
    return DEER_OK;
}

int deer_prefill(deer_ctx *c, int32_t batch, const int32_t *ids, const int32_t *lens) {
    if (!c) return DEER_EINVAL;
    if (!ids || !lens || batch < 1 || batch > c->p.max_batch) return fail(c, DEER_EINVAL, "bad batch or null pointer");
    for (int b = 0; b < batch; ++b) {
        if (lens[b] < 1) return fail(c, DEER_EINVAL, "prompt %d is empty", b);
        if (lens[b] + c->p.max_k > c->p.max_seq) return fail(c, DEER_ECAPACITY, "prompt %d: %d tokens + one block exceed max_seq %d", b, lens[b], c->p.max_seq);
    }
    std::vector<int> pend(batch), lenv(lens, lens + batch);
    std::vector<size_t> offs(batch);
    size_t total = 0;
    for (int b = 0; b < batch; ++b) {
        offs[b] = total;
        for (int i = 0; i < lens[b]; ++i)
            if (ids[total + i] < 0 || ids[total + i] >= c->p.target.vocab) return fail(c, DEER_EINVAL, "token id outside the vocabulary");
        total += lens[b];
        pend[b] = ids[total - 1];
    }
    // Passes of up to cap attention tiles, each up to 32 rows of one sequence; a pass takes the next tiles of as many sequences
    // as fit, and its GEMM rows follow each other without gaps (rows of one sequence that are split over passes continue in
    // the next pass, over the keys the earlier pass has written).  The buffers hold PREFILL_TILES tiles, and what a draft pass
    // of max_batch sequences needs: many short prompts of a large batch then go through in fewer passes.
    const int cap = c->max_tiles;
    std::vector<PrefillPass> passes[2];
    for (int model = 0; model < 2; ++model)
        for (int b = 0; b < batch; ++b) {
            const int nrows = (model == DEER_TARGET) ? lens[b] - 1 : lens[b];   // the last token stays pending for the target
            for (int c0 = 0; c0 < nrows;) {
                std::vector<PrefillPass> &ps = passes[model];
                if (ps.empty() || (int)ps.back().desc.size() == cap) ps.emplace_back();
                PrefillPass &pa = ps.back();
                const int take = std::min(nrows - c0, 32);
                pa.desc.push_back(make_int4(b, c0, take | pa.n_rows << 6, (int)(offs[b] + c0)));
                pa.maxlim = std::max(pa.maxlim, c0 + take);
                c0 += take;
                pa.n_rows += take;
            }
        }
    c->state = ST_INIT;   // no sequences until all of the call has worked: the device state may be of the new ones, the host's of the old
    int rc = enqueue_prefill(c, batch, ids, lens, pend.data(), total, passes);
    if (rc && c->side) (void)hipStreamSynchronize(c->side);   // (without an error the library's stream waits for it)
    const hipError_t e = hipStreamSynchronize(c->stream);   // after an error too: the next call writes to the same staging memory
    if (rc) return rc;
    if (e != hipSuccess) return fail(c, DEER_EHIP, "prefill: %s", hipGetErrorString(e));
    set_state(c, batch, lenv.data());
    return DEER_OK;
}

int deer_set_prefilled(deer_ctx *c, int32_t batch, const int32_t *lens, const int32_t *last) {
    if (!c) return DEER_EINVAL;
    if (!lens || !last || batch < 1 || batch > c->p.max_batch) return fail(c, DEER_EINVAL, "bad batch or null pointer");
    for (int b = 0; b < batch; ++b) {
        if (lens[b] < 1) return fail(c, DEER_EINVAL, "sequence %d is empty", b);
        if (lens[b] + c->p.max_k > c->p.max_seq) return fail(c, DEER_ECAPACITY, "sequence %d exceeds max_seq", b);
        if (last[b] < 0 || last[b] >= c->p.target.vocab) return fail(c, DEER_EINVAL, "token id outside the vocabulary");
    }
    const size_t bytes = c->wk.up_desc;
    char *img = upload_image(c, bytes);
    fill_state(c, img, batch, lens, lens, last);
    c->state = ST_INIT;   // (see deer_prefill)
    const hipError_t e = hipMemcpyAsync(c->wk.up, img, bytes, hipMemcpyHostToDevice, c->stream), e2 = hipStreamSynchronize(c->stream);
    if (e != hipSuccess || e2 != hipSuccess) return fail(c, DEER_EHIP, "state: %s", hipGetErrorString(e != hipSuccess ? e : e2));
    set_state(c, batch, lens);
    return DEER_OK;
}

int deer_draft_block_multipass(deer_ctx *c, int32_t k, float T, uint64_t seed, int32_t n_passes, int32_t *draft_dev) {
    if (!c) return DEER_EINVAL;
    if (!draft_dev || k < 1 || k > c->p.max_k || !(T >= 0.f)) return fail(c, DEER_EINVAL, "bad k, T or null pointer");
    if (n_passes < 1 || n_passes > k) return fail(c, DEER_EINVAL, "n_passes must be in 1..k");
    if (c->state != ST_PREFILLED) return fail(c, DEER_ESTATE, "draft_block needs a prefilled or committed state");
    if (k + c->bonus > 32) return fail(c, DEER_EINVAL, "with the bonus token on, k must be at most 31 (k + 1 rows per tile)");
    const int B = c->batch;
    int maxlim = 0, n_ing = 0, max_ing = 0;
    for (int b = 0; b < B; ++b) {
        if (c->h_len[b] + k > c->p.max_seq) return fail(c, DEER_ECAPACITY, "sequence %d: length %d + k exceeds max_seq", b, c->h_len[b]);
        maxlim = std::max(maxlim, c->h_len[b] + k);
        n_ing += c->h_ing_n[b];
        max_ing = std::max(max_ing, c->h_ing_n[b]);
    }
    Work &w = c->wk;
    double keys = 0;
    for (int b = 0; b < B; ++b) keys += c->h_len[b] + k;
    // pass s fixes block positions [lo, hi), lo = ceil(k (s-1) / n), hi = ceil(k s / n); the first pass also
    // ingests the committed tokens the drafter has not cached yet
    for (int s = 1; s <= n_passes; ++s) {
        const int lo = (k * (s - 1) + n_passes - 1) / n_passes, hi = (k * s + n_passes - 1) / n_passes;
        if (hi == lo) continue;
        PassRows pr{};
        pr.kind = ROWS_DRAFT; pr.st = w.st; pr.tokens = draft_dev; pr.k = k; pr.nrows = 0; pr.vocab = c->p.drafter.vocab;
        pr.mask_id = c->p.mask_token_id; pr.n_fixed = lo; pr.B = B; pr.n_ingest = n_ing; pr.share = k + max_ing <= 32;
        LmPlan lm{true, B * k, k, T, seed, lo, T > 0.f, draft_dev};
        int rc = run_pass(c, DEER_DRAFTER, (B * k + n_ing + 31) / 32, n_ing > 0 && !pr.share ? 2 * B : B, maxlim, lm, keys, pr);
        if (rc) return rc;
        n_ing = max_ing = 0;   // the device-side counts were cleared by k_rowstat_final
    }
    std::fill(c->h_ing_n.begin(), c->h_ing_n.end(), 0);
    c->cur_k = k;
    c->cur_T = T;
    c->state = ST_DRAFTED;
    return DEER_OK;
}

int deer_draft_block(deer_ctx *c, int32_t k, float T, uint64_t seed, int32_t *draft_dev) {
    return deer_draft_block_multipass(c, k, T, seed, 1, draft_dev);
}

int deer_verify_block(deer_ctx *c, int32_t k, float T, const int32_t *draft_dev) {
    if (!c) return DEER_EINVAL;
    if (!draft_dev || k < 1 || k > c->p.max_k || !(T >= 0.f)) return fail(c, DEER_EINVAL, "bad k, T or null pointer");
    if (c->state != ST_DRAFTED) return fail(c, DEER_ESTATE, "verify_block must follow draft_block");
    if (k != c->cur_k || T != c->cur_T) return fail(c, DEER_EINVAL, "k and T must match the draft_block call");
    const int B = c->batch;
    const int nrows = k + c->bonus;   // [x_j, y^_1 .. y^_{k-1}] and, with the bonus token, y^_k
    int maxlim = 0;
    for (int b = 0; b < B; ++b) maxlim = std::max(maxlim, c->h_len[b] - 1 + nrows);
    Work &w = c->wk;
    PassRows pr{};
    pr.kind = ROWS_VERIFY; pr.st = w.st; pr.tokens = draft_dev; pr.k = k; pr.nrows = nrows; pr.vocab = c->p.target.vocab;
    pr.B = B;
    LmPlan lm{true, B * nrows, nrows, T, 0};
    double keys = 0;
    for (int b = 0; b < B; ++b) keys += c->h_len[b] - 1 + nrows;
    int rc = run_pass(c, DEER_TARGET, (B * nrows + 31) / 32, B, maxlim, lm, keys, pr);
    if (rc) return rc;
    c->wk_draft = draft_dev;
    c->state = ST_VERIFIED;
    return DEER_OK;
}

// Shared by the two acceptance entry points: acc_part / acc_cnt are the sampling kernel's scratch (from the
// caller's workspace, or the library's static array).
static int accept_impl(deer_ctx *c, int32_t k, float T, uint64_t seed, int32_t *acc, int32_t *committed, int32_t *ncom,
                       AccPart *acc_part, int *acc_cnt, bool no_alloc) {
    if (!acc || !committed || !ncom || k < 1 || k > c->p.max_k || !(T >= 0.f)) return fail(c, DEER_EINVAL, "bad k, T or null pointer");
    if (c->state != ST_VERIFIED) return fail(c, DEER_ESTATE, "accept_and_commit must follow verify_block");
    if (k != c->cur_k || T != c->cur_T) return fail(c, DEER_EINVAL, "k and T must match the draft_block call");
    const int B = c->batch;
    Work &w = c->wk;
    const int V = c->p.target.vocab;
    const int cs = k + c->bonus;   // committed tokens per sequence: at most k, or k + 1 with the bonus token
    const char *d0 = (const char *)w.ao.accept_len;
    const size_t o_n = (const char *)w.ao.n_committed - d0, o_c = (const char *)w.ao.committed - d0;
    const size_t bytes = o_c + (size_t)B * cs * 4;
    char *host = c->h_pin;
    if (!host || bytes > c->h_pin_bytes) {
        if (no_alloc) return fail(c, DEER_ECAPACITY, "no page-locked result buffer was set up at init");
        c->h_ao.resize(bytes);
        host = c->h_ao.data();
    }
    // the kernels write their few results straight into page-locked host memory where there is some (a copy behind them is one
    // more launch of a few microseconds per iteration)
    const bool direct = host == c->h_pin && c->h_pin_dev;
    AcceptOut ao = w.ao;
    if (direct) ao = AcceptOut{(int *)c->h_pin_dev, (int *)(c->h_pin_dev + o_n), (int *)(c->h_pin_dev + o_c)};
    if (T == 0.f)
        hipLaunchKernelGGL(k_accept_greedy, dim3(B), dim3(64), 0, c->stream, w.st, ao, c->wk_draft, w.res[DEER_TARGET], k,
                           c->p.eos_token_id, c->bonus);
    else
        hipLaunchKernelGGL(k_accept_sample, dim3(B, ACC_NB), dim3(1024), 0, c->stream, w.st, ao, c->wk_draft, w.res[DEER_TARGET],
                           w.res[DEER_DRAFTER], w.logits[DEER_TARGET], w.logits[DEER_DRAFTER], k, V, T, seed, c->p.eos_token_id,
                           c->bonus, acc_part, acc_cnt, w.rm.pos);
    LAUNCHCHK(c, "k_accept");
    // (the three result arrays lie one after the other in the workspace: one copy)
    if (!direct) HIPCHK(c, hipMemcpyAsync(host, d0, bytes, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    memcpy(acc, host, (size_t)B * 4);
    memcpy(ncom, host + o_n, (size_t)B * 4);
    memcpy(committed, host + o_c, (size_t)B * cs * 4);
    for (int b = 0; b < B; ++b) {
        c->h_len[b] += ncom[b];
        c->h_ing_n[b] = ncom[b];
        if (c->p.eos_token_id >= 0 && ncom[b] > 0 && committed[(size_t)b * cs + ncom[b] - 1] == c->p.eos_token_id) c->h_finished[b] = 1;
    }
    c->state = ST_PREFILLED;
    return DEER_OK;
}

int deer_accept_and_commit(deer_ctx *c, int32_t k, float T, uint64_t seed, int32_t *acc, int32_t *committed, int32_t *ncom) {
    if (!c) return DEER_EINVAL;
    return accept_impl(c, k, T, seed, acc, committed, ncom, c->wk.acc_part, c->wk.acc_cnt, false);
}

int deer_accept_and_commit_static(deer_ctx *c, int32_t k, float T, uint64_t seed, int32_t *acc, int32_t *committed, int32_t *ncom) {
    if (!c) return DEER_EINVAL;
    if (c->batch > STATIC_MAX_BATCH) return fail(c, DEER_ECAPACITY, "the static scratch holds %d sequences, the batch has %d", STATIC_MAX_BATCH, c->batch);
    if (!c->static_scratch) return fail(c, DEER_EHIP, "the static scratch was not resolved for device %d", c->p.device);
    AccPart *part = (AccPart *)c->static_scratch;
    int *cnt = (int *)((char *)c->static_scratch + STATIC_PART_BYTES);
    if (T > 0.f && c->state == ST_VERIFIED) {
        // the array keeps the last call's contents: the arrival counters of this batch start at zero (a fill kernel,
        // not a memset node); stale candidates are overwritten before the last arrival reads them
        hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(STATIC_MAX_BATCH), 0, c->stream, (uint32_t *)cnt, 0u, (size_t)c->batch);
        LAUNCHCHK(c, "k_fill_u32");
    }
    return accept_impl(c, k, T, seed, acc, committed, ncom, part, cnt, true);
}

int deer_set_bonus_token(deer_ctx *c, int enable) {
    if (!c) return DEER_EINVAL;
    if (c->state == ST_DRAFTED || c->state == ST_VERIFIED) return fail(c, DEER_ESTATE, "the bonus token cannot change inside an iteration");
    c->bonus = enable ? 1 : 0;
    return DEER_OK;
}

int deer_destroy(deer_ctx *c) {
    if (!c) return DEER_EINVAL;
    (void)hipStreamSynchronize(c->stream);
    for (hipEvent_t e : c->ev_pool) (void)hipEventDestroy(e);
    if (c->side) { (void)hipStreamSynchronize(c->side); (void)hipStreamDestroy(c->side); }
    if (c->fork) (void)hipEventDestroy(c->fork);
    if (c->join) (void)hipEventDestroy(c->join);
    if (c->h_pin) (void)hipHostFree(c->h_pin);
    if (c->h_up) (void)hipHostFree(c->h_up);
    delete c;
    return DEER_OK;
}

const char *deer_last_error(const deer_ctx *c) { return c ? c->err.c_str() : g_init_error.c_str(); }

int deer_debug_get_logits(deer_ctx *c, int model, float *out, size_t n_floats) {
    if (!c) return DEER_EINVAL;
    if (!out || model < 0 || model > 1) return fail(c, DEER_EINVAL, "bad model or null pointer");
    if (c->cur_k < 1) return fail(c, DEER_ESTATE, "no pass has run yet");
    if (!c->p.keep_logits && c->cur_T == 0.f) return fail(c, DEER_ESTATE, "logits were not kept (keep_logits = 0 and T = 0)");
    const size_t n = (size_t)c->batch * (c->cur_k + (model == DEER_TARGET ? c->bonus : 0)) * c->p.target.vocab;
    if (n_floats < n) return fail(c, DEER_ECAPACITY, "output holds %zu floats, need %zu", n_floats, n);
    HIPCHK(c, hipMemcpyAsync(out, c->wk.logits[model], n * 4, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    return DEER_OK;
}

int deer_debug_profile(deer_ctx *c, int enable) {
    if (!c) return DEER_EINVAL;
    prof_close(c);
    HIPCHK(c, hipStreamSynchronize(c->stream));
    c->prof_on = enable != 0;
    c->prof.clear();
    c->ev_used = 0;
    return DEER_OK;
}

int deer_debug_profile_read(deer_ctx *c, int kernel_class, double *total_ms, int64_t *launches, double *bytes) {
    if (!c || !total_ms || !launches || !bytes) return DEER_EINVAL;
    prof_close(c);
    HIPCHK(c, hipStreamSynchronize(c->stream));
    *total_ms = 0.0; *launches = 0; *bytes = 0.0;
    for (const auto &r : c->prof) {
        if (r.cls != kernel_class) continue;
        float ms = 0.f;
        HIPCHK(c, hipEventElapsedTime(&ms, r.a, r.b));
        *total_ms += ms; *launches += r.launches; *bytes += r.bytes;
    }
    return DEER_OK;
}

int deer_debug_gemm_stamps(deer_ctx *c, int model, int launch, uint64_t *stamps_host, int32_t max_blocks, int32_t *blocks) {
    if (!c) return DEER_EINVAL;
    if (model < 0 || model > 1) return fail(c, DEER_EINVAL, "bad model");
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if (blocks) *blocks = c->stamp_blocks;
    if (stamps_host && c->stamp_blocks > 0 && max_blocks > 0)
        HIPCHK(c, hipMemcpy(stamps_host, c->wk.stamps, (size_t)std::min(max_blocks, c->stamp_blocks) * 64, hipMemcpyDeviceToHost));
    c->stamp_model = model;
    c->stamp_launch = launch;
    c->stamp_blocks = 0;
    return DEER_OK;
}

int deer_debug_route_spread(deer_ctx *c, int enable) {
    if (!c) return DEER_EINVAL;
    c->route_spread = enable ? 1 : 0;
    return DEER_OK;
}

int deer_debug_experts_streamed(deer_ctx *c, int64_t *pairs) {
    if (!c || !pairs) return DEER_EINVAL;
    *pairs = 0;
    if (!c->wk.moe_touched) return DEER_OK;
    unsigned long long v = 0;
    HIPCHK(c, hipStreamSynchronize(c->stream));
    HIPCHK(c, hipMemcpy(&v, c->wk.moe_touched, 8, hipMemcpyDeviceToHost));
    HIPCHK(c, hipMemset(c->wk.moe_touched, 0, 8));
    *pairs = (int64_t)v;
    return DEER_OK;
}

int deer_debug_stream_read(deer_ctx *c, const void *buf_dev, size_t bytes, int32_t workgroups, int32_t nontemporal,
                           int32_t reps, float *ms_per_read) {
    if (!c || !ms_per_read) return DEER_EINVAL;
    if (!buf_dev || bytes < 16 || bytes % 16 || ((uintptr_t)buf_dev & 15)) return fail(c, DEER_EINVAL, "buffer must be 16-byte aligned, a multiple of 16 bytes");
    if (workgroups < 1 || workgroups > (1 << 20) || reps < 1 || reps > 10000) return fail(c, DEER_EINVAL, "bad workgroups / reps");
    if (c->prof_on) return fail(c, DEER_ESTATE, "launch timing is on");
    uint32_t *out = (uint32_t *)c->wk.stamps;   // a word of the debugging buffer
    const size_t n = bytes / 16;
    auto launch = [&]() {
        if (nontemporal) hipLaunchKernelGGL(k_stream_read<true>, dim3((unsigned)workgroups), dim3(512), 0, c->stream, (const u32x4 *)buf_dev, n, out);
        else hipLaunchKernelGGL(k_stream_read<false>, dim3((unsigned)workgroups), dim3(512), 0, c->stream, (const u32x4 *)buf_dev, n, out);
    };
    for (int i = 0; i < 3; ++i) launch();
    LAUNCHCHK(c, "k_stream_read");
    hipEvent_t e0 = prof_event(c), e1 = prof_event(c);
    if (!e0 || !e1) return fail(c, DEER_EHIP, "hipEventCreate failed");
    HIPCHK(c, hipEventRecord(e0, c->stream));
    for (int i = 0; i < reps; ++i) launch();
    HIPCHK(c, hipEventRecord(e1, c->stream));
    HIPCHK(c, hipEventSynchronize(e1));
    float ms = 0.f;
    HIPCHK(c, hipEventElapsedTime(&ms, e0, e1));
    c->ev_used -= 2;   // the two events go back to the pool
    *ms_per_read = ms / (float)reps;
    return DEER_OK;
}

int deer_debug_gemm_tiled(deer_ctx *c, int min_tiles) {
    if (!c) return DEER_EINVAL;
    if (min_tiles < 0) return fail(c, DEER_EINVAL, "min_tiles must not be negative");
    c->block_gemm = min_tiles;
    c->slim = min_tiles != 0;
    return DEER_OK;
}

int deer_debug_gemm_block(deer_ctx *c, int nb, int ring, int splits) {
    if (!c) return DEER_EINVAL;
    if (nb != 0 && !((nb == 2 && (ring == 4 || ring == 8)) || (nb == 4 && ring == 4))) return fail(c, DEER_EINVAL, "no such form of the blocked GEMM");
    if (nb != 0 && (splits < 1 || splits > 8)) return fail(c, DEER_EINVAL, "splits must be in 1..8");
    c->force_nb = nb; c->force_ring = ring; c->force_S = splits;
    return DEER_OK;
}

int deer_debug_force_commit(deer_ctx *c, const int32_t *tokens, const int32_t *n, int32_t stride) {
    if (!c) return DEER_EINVAL;
    if (!tokens || !n || stride < 1) return fail(c, DEER_EINVAL, "null pointer or bad stride");
    if (c->state != ST_VERIFIED) return fail(c, DEER_ESTATE, "force_commit stands in for accept_and_commit: it must follow verify_block");
    const int B = c->batch, cs = c->cur_k + c->bonus;
    if (stride > 32) return fail(c, DEER_EINVAL, "stride must be at most 32");
    for (int b = 0; b < B; ++b) {
        if (n[b] < 0 || n[b] > cs || n[b] > stride) return fail(c, DEER_EINVAL, "sequence %d: %d tokens, at most %d fit this block", b, n[b], std::min(cs, stride));
        for (int i = 0; i < n[b]; ++i)
            if (tokens[(size_t)b * stride + i] < 0 || tokens[(size_t)b * stride + i] >= c->p.target.vocab) return fail(c, DEER_EINVAL, "token id outside the vocabulary");
    }
    Work &w = c->wk;
    // staged through the acceptance result arrays (unused until the next accept_and_commit)
    HIPCHK(c, hipMemcpyAsync(w.ao.committed, tokens, (size_t)B * stride * 4, hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipMemcpyAsync(w.ao.n_committed, n, (size_t)B * 4, hipMemcpyHostToDevice, c->stream));
    hipLaunchKernelGGL(k_force_commit, dim3((B + 63) / 64), dim3(64), 0, c->stream, w.st, w.ao.committed, w.ao.n_committed, stride,
                       c->p.eos_token_id, B);
    LAUNCHCHK(c, "k_force_commit");
    HIPCHK(c, hipStreamSynchronize(c->stream));   // the host arrays may be reused by the caller
    for (int b = 0; b < B; ++b) {
        c->h_len[b] += n[b];
        c->h_ing_n[b] = n[b];
        for (int i = 0; i < n[b]; ++i)
            if (c->p.eos_token_id >= 0 && tokens[(size_t)b * stride + i] == c->p.eos_token_id) c->h_finished[b] = 1;
    }
    c->state = ST_PREFILLED;
    return DEER_OK;
}

int deer_debug_load_kv(deer_ctx *c, int model, int32_t layer, int32_t seq, int32_t first_slot, int32_t n_slots,
                       const void *k_rows_dev, const void *v_rows_dev) {
    if (!c) return DEER_EINVAL;
    if (model < 0 || model > 1 || !k_rows_dev || !v_rows_dev) return fail(c, DEER_EINVAL, "bad model or null pointer");
    ModelRT &m = c->m[model];
    if (layer < 0 || layer >= m.c.n_layers || seq < 0 || seq >= c->p.max_batch) return fail(c, DEER_EINVAL, "layer or sequence out of range");
    if (first_slot < 0 || n_slots < 0 || (int64_t)first_slot + n_slots > c->p.max_seq) return fail(c, DEER_ECAPACITY, "slots %d .. %d exceed max_seq %d", first_slot, first_slot + n_slots, c->p.max_seq);
    if (n_slots == 0) return DEER_OK;
    const KvView kv{m.kv + m.kv_k_base + (size_t)layer * m.kv_layer_stride, m.kv + m.kv_v_base + (size_t)layer * m.kv_layer_stride,
                    m.kv_seq_stride, m.kv_head_stride, c->p.max_seq};
    const size_t items = (size_t)n_slots * m.c.n_kv_heads * (m.c.head_dim / 8);
    hipLaunchKernelGGL(k_load_kv, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, c->stream, (const uint16_t *)k_rows_dev,
                       (const uint16_t *)v_rows_dev, kv, seq, first_slot, n_slots, m.c.n_kv_heads, m.c.head_dim);
    LAUNCHCHK(c, "k_load_kv");
    return DEER_OK;
}

int deer_get_lengths(const deer_ctx *c, int32_t *len) {
    if (!c || !len) return DEER_EINVAL;
    for (int b = 0; b < c->batch; ++b) len[b] = c->h_len[b];
    return DEER_OK;
}

int deer_get_kv_layout(const deer_ctx *c, int model, deer_kv_layout *out) {
    if (!c || !out || model < 0 || model > 1) return DEER_EINVAL;
    const ModelRT &m = c->m[model];
    out->k_base = m.kv_k_base; out->v_base = m.kv_v_base;
    out->layer_stride = m.kv_layer_stride; out->seq_stride = m.kv_seq_stride; out->head_stride = m.kv_head_stride;
    out->max_seq = c->p.max_seq; out->head_dim = m.c.head_dim;
    return DEER_OK;
}

}  // extern "C"
