"""Performance cases of the draft-verify library: what a serving program has it do, through DeerEngine.

A case is one of three kinds of call sequence:
  prefill   a batch of prompts enters: both KV caches are built (deer_prefill).
  decode    iterations of draft -> verify -> accept from a state with a given prefix length per sequence; the second
            iteration of a case (iters = 2) also has the drafter take in the tokens that the first one committed, as
            every iteration of a running loop does.
  request   prefill and one iteration: a short request from its prompt to its first tokens, also what a program
            without a kept KV cache does for every block.
Shapes are the ones the library is used with (Qwen3 4B and 8B, the 30B-A3B mixture, the 24-layer 0.5B drafter, and the
tiny pair of the tests).  Where a case has fewer layers than the model, target and drafter are shortened in the same
proportion: the launches of a layer are the same, and a 64-bit reference of the case stays affordable.

Weights are N(0, 0.02^2) in bf16 and unit RMSNorm gains; stand-in cache rows are N(0, 1), the scale that such a model's K
and V rows have.  The mixture's embeddings are N(0, 1): its rows then stay different from layer to layer and the router
spreads them over the experts as a trained one does (with 0.02 every row of a block ends up on the same few).

The verify pass is given a fixed random block instead of the drafter's tokens: random weights leave argmax margins so
small that one rounding somewhere in the drafter would change what the target is asked, and with it every later output.
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

from paper_2512_15176_amd.binding import DEER_DRAFTER, DEER_TARGET, DeerEngine


@dataclasses.dataclass(frozen=True)
class Shape:
    n_layers: int
    d_model: int
    n_q_heads: int
    n_kv_heads: int
    head_dim: int
    d_ff: int
    vocab: int
    n_experts: int = 0
    top_k: int = 0
    d_ff_expert: int = 0
    rope_base: float = 1e6
    rms_eps: float = 1e-6

    def dims(self, name):
        d, q, kv = self.d_model, self.n_q_heads * self.head_dim, self.n_kv_heads * self.head_dim
        f = self.d_ff_expert if self.n_experts else self.d_ff
        return {"embed": (self.vocab, d), "lm_head": (d, self.vocab), "wq": (d, q), "wk": (d, kv), "wv": (d, kv),
                "wo": (q, d), "wg": (d, f), "wu": (d, f), "wd": (f, d), "router": (d, self.n_experts)}[name]


DRAFTER = Shape(24, 896, 14, 2, 64, 4864, 151936)
MODELS = {   # target, drafter
    "tiny": (Shape(2, 128, 4, 2, 32, 512, 1024, rope_base=10000.0), Shape(1, 128, 4, 2, 32, 512, 1024, rope_base=10000.0)),
    "4b": (Shape(36, 2560, 32, 8, 128, 9728, 151936), DRAFTER),
    "8b": (Shape(36, 4096, 32, 8, 128, 12288, 151936), DRAFTER),
    "a3b": (Shape(48, 2048, 32, 4, 128, 0, 151936, n_experts=128, top_k=8, d_ff_expert=768), DRAFTER),
}
SHORT = {"tiny": (2, 1), "4b": (12, 8), "8b": (12, 8), "a3b": (8, 4)}   # layers of the shortened pairs


def _case(name, kind, model, batch, lo, hi, layers=None, k=32, T=0.0, iters=1, bonus=False):
    """lo .. hi: the sequences' lengths (prompt or prefix) are spread over this range."""
    t, d = layers or SHORT[model]
    c = {"kind": kind, "model": model, "layers": t, "drafter_layers": d, "batch": batch, "lo": lo, "hi": hi}
    if kind != "prefill":
        c.update({"k": k, "T": T, "iters": iters, "bonus": bonus})
    return dict({"name": name}, **c) if name else c


def listed():
    return [
        # the smallest call: a 64-token prompt to the first block, a few launches of a few microseconds each
        _case("tiny_request", "request", "tiny", 1, 64, 64, k=8),
        # one short prompt (a function signature with its docstring), full depth: time to the first block
        _case("prefill_4b_short", "prefill", "4b", 1, 201, 201, layers=(36, 24)),
        # prompts of different lengths that arrive together
        _case("prefill_4b_batch", "prefill", "4b", 8, 60, 700),
        # the benchmark's prefill: a 4096-token context, full depth
        _case("prefill_8b_4096", "prefill", "8b", 1, 4096, 4096, layers=(36, 24)),
        # the mixture's prefill
        _case("prefill_a3b_2048", "prefill", "a3b", 1, 2048, 2048),
        # the benchmark's decoding loop: one sequence, greedy, blocks of 32, full depth
        _case("decode_8b", "decode", "8b", 1, 4096, 4096, layers=(36, 24), iters=2),
        # one sequence of the smaller target with sampling, shorter blocks and the bonus token, full depth
        _case("decode_4b_sample", "decode", "4b", 1, 1023, 1023, layers=(36, 24), k=16, T=0.6, bonus=True),
        # a small batch of unequal sequences, greedy, blocks of 16
        _case("decode_8b_b4", "decode", "8b", 4, 200, 1500, k=16, iters=2),
        # a large batch, sampling
        _case("decode_8b_b16", "decode", "8b", 16, 512, 2048, T=1.0),
        # the mixture's decoding loop
        _case("decode_a3b", "decode", "a3b", 1, 2048, 2048, iters=2),
        # the mixture under a small batch, sampling
        _case("decode_a3b_b8", "decode", "a3b", 8, 300, 1200, k=16, T=0.6),
        # sixteen long contexts: bound by the caches
        _case("decode_8b_long_b16", "decode", "8b", 16, 32768, 32768, layers=(6, 4), T=1.0),
    ]


def draw(rng):
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["prefill", "prefill", "prefill", "decode", "decode", "decode", "decode", "request"])
    model = rng.choice(["4b", "8b", "a3b"]) if rng.random() < 0.9 else "tiny"
    k = rng.randint(1, 32)
    T = rng.choice([0.0, 0.0, 0.6, 1.0])
    bonus = k < 32 and rng.random() < 0.25
    if kind == "decode":
        batch = spread(1, 16)
        hi = spread(32, 8192 if batch <= 8 else 4096)
        return _case(None, kind, model, batch, max(1, int(hi * rng.uniform(0.25, 1.0))), hi, k=k, T=T,
                     iters=2 if T == 0.0 else 1, bonus=bonus)
    batch = spread(1, 8)
    hi = max(8, spread(16, 4096) // batch)
    return _case(None, kind, model, batch, max(2, int(hi * rng.uniform(0.25, 1.0))), hi, k=k, T=T, bonus=bonus)


# ------------------------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------------------------
def _shapes(case):
    t, d = MODELS[case["model"]]
    return dataclasses.replace(t, n_layers=case["layers"]), dataclasses.replace(d, n_layers=case["drafter_layers"])


def _lens(case):
    """Lengths spread evenly over lo .. hi, in no particular order."""
    lo, hi = case["lo"], case["hi"]
    return [lo + int((hi - lo + 1) * ((0.5 + 0.6180339887 * b) % 1.0)) if hi > lo else hi for b in range(case["batch"])]


def _max_seq(case):
    return -(-(max(_lens(case)) + 32 + 33 * case.get("iters", 0)) // 64) * 64


def _rng(*key):
    x = 0
    for v in key:
        x = (x * 1000003 + v + 1) % (1 << 61)
    return torch.Generator(device="cuda").manual_seed(x)


NAMES = ("embed", "lm_head", "wq", "wk", "wv", "wo", "router", "wg", "wu", "wd")


def _weights(shape, seed, model, name, layer=-1):
    """bf16 [rows][cols], or [experts][rows][cols] of a mixture's expert tensors."""
    dims = shape.dims(name)
    if shape.n_experts and name in ("wg", "wu", "wd"):
        dims = (shape.n_experts,) + dims
    w = torch.randn(dims, generator=_rng(seed, model, NAMES.index(name), layer), device="cuda", dtype=torch.bfloat16)
    return w if name == "embed" and shape.n_experts else w.mul_(0.02)


def _layer_names(shape):
    return ("wq", "wk", "wv", "wo") + (("router",) if shape.n_experts else ()) + ("wg", "wu", "wd")


def _cache_rows(shape, seed, model, layer, lens):
    """Per sequence: stand-in K and V rows [len][kv_head][head_dim]."""
    g = _rng(seed, model, 77, layer)
    return [tuple(torch.randn(n, shape.n_kv_heads, shape.head_dim, generator=g, device="cuda", dtype=torch.bfloat16) for _ in "kv")
            for n in lens]


def _tokens(case, seed):
    """Prompts (prefill, request) or last tokens (decode), and the blocks that the verify passes are given."""
    r = np.random.default_rng([seed, 5])
    vocab = MODELS[case["model"]][0].vocab
    prompts = [r.integers(0, vocab, n).astype(np.int32) for n in (_lens(case) if case["kind"] != "decode" else [1] * case["batch"])]
    blocks = r.integers(0, vocab, (case.get("iters", 0), case["batch"], case.get("k", 1))).astype(np.int32)
    return prompts, blocks


class State:
    pass


def _find_logits(s):
    """The engine keeps a pass's logits in the workspace, which the caller owns; debug_get_logits copies them to the
    host, which no serving program waits for.  Finds where they lie by the values of a pass with k = 1."""
    eng, T = s.eng, s.case["T"]
    eng.set_prefilled([1] * s.case["batch"], [p[-1] for p in s.prompts])
    eng.draft_block(1, T, 0)
    eng.verify_block(1, T, s.blocks[0][:, :1].contiguous())
    words = eng._workspace[: eng._workspace.numel() // 4 * 4].view(torch.int32)
    views = []
    for model in (DEER_DRAFTER, DEER_TARGET):
        want = torch.from_numpy(eng.debug_get_logits(model, 1).reshape(-1)[:256].copy()).view(torch.int32).cuda()
        at = [i for i in (words[:-256] == want[0]).nonzero().flatten().tolist() if bool((words[i : i + 256] == want).all())]
        assert at, "the logits were not found in the workspace"   # the first: empty caches give every sequence the same row
        rows = s.case["k"] + (s.case["bonus"] if model == DEER_TARGET else 0)
        n = s.case["batch"] * rows * eng.target.vocab
        views.append(words[at[0] : at[0] + n].view(torch.float32).view(s.case["batch"], rows, eng.target.vocab))
    return views


def _cache_view(eng, model, shape):
    """The caller-owned cache as [K, V][layer][sequence][kv head][32-slot block][fragment][lane][8]."""
    lay = eng.get_kv_layout(model)
    assert lay.k_base == 0 and lay.v_base == shape.n_layers * lay.layer_stride and lay.seq_stride == shape.n_kv_heads * lay.head_stride
    n = 2 * shape.n_layers * lay.layer_stride
    return eng._kv[model][: 2 * n].view(torch.bfloat16).view(2, shape.n_layers, eng.max_batch, shape.n_kv_heads,
                                                              lay.max_seq // 32, shape.head_dim // 16, 64, 8)


def _new_blocks(case, b):
    """The 32-slot blocks of sequence b that a case's verify passes write to."""
    n = _lens(case)[b] - 1
    return slice(n // 32, (n + case["iters"] * (case["k"] + case["bonus"]) + 31) // 32)


def prepare(case, seed):
    s = State()
    s.case, s.lens = case, _lens(case)
    shapes = _shapes(case)
    decode = case["kind"] != "prefill"
    s.eng = DeerEngine(*shapes, case["batch"], _max_seq(case), 32, shapes[0].vocab - 1, keep_logits=decode)
    for model, shape in enumerate(shapes):
        for layer in range(-1, shape.n_layers):
            for name in ("embed", "lm_head") if layer < 0 else _layer_names(shape):
                w = _weights(shape, seed, model, name, layer)
                for e, x in enumerate(w) if w.dim() == 3 else [(-1, w)]:
                    s.eng.load_tensor(model, name, layer, e, x)
    s.prompts, blocks = _tokens(case, seed)
    if decode:
        s.blocks = list(torch.from_numpy(blocks).cuda())
        s.last = [int(p[-1]) for p in s.prompts]
        s.draft_logits, s.verify_logits = _find_logits(s)
        if case["bonus"]:
            s.eng.set_prefilled(s.lens, s.last)   # the option changes between iterations only
            s.eng.set_bonus_token(True)
        if case["kind"] == "decode":
            for model, shape in enumerate(shapes):
                for layer in range(shape.n_layers):
                    for b, (k, v) in enumerate(_cache_rows(shape, seed, model, layer, s.lens)):
                        s.eng.debug_load_kv(model, layer, b, 0, k, v)
        view = _cache_view(s.eng, DEER_TARGET, shapes[0])
        s.new_kv = [view[:, :, b, :, _new_blocks(case, b)] for b in range(case["batch"])]
    else:
        s.caches = [_cache_view(s.eng, m, shapes[m]) for m in (DEER_TARGET, DEER_DRAFTER)]
    torch.cuda.synchronize()
    return s


def run(s):
    c, eng = s.case, s.eng
    if c["kind"] == "decode":
        eng.set_prefilled(s.lens, s.last)
    else:
        eng.prefill(s.prompts)
        if c["kind"] == "prefill":
            return {"target_cache": s.caches[0], "drafter_cache": s.caches[1]}
    k, T = c["k"], c["T"]
    for block in s.blocks:
        eng.draft_block(k, T, 4)
        eng.verify_block(k, T, block)
        accepted, committed, n = eng.accept_and_commit(k, T, 4)
    tokens = np.full((c["batch"], k + 1), -1, np.int32)
    for b, t in enumerate(committed):
        tokens[b, : len(t)] = t
    return {"draft_logits": s.draft_logits, "verify_logits": s.verify_logits, "accepted": accepted, "committed": tokens,
            "new_cache_rows": s.new_kv}


# ------------------------------------------------------------------------------------------------------------------
# work and tolerance
# ------------------------------------------------------------------------------------------------------------------
def _pass_work(shape, rows, keys, logit_rows):
    """rows: token rows; keys: (visible keys, cached keys read) summed over rows and over sequences."""
    d, hd, q, kv = shape.d_model, shape.head_dim, shape.n_q_heads, shape.n_kv_heads
    attn = d * (q + 2 * kv) * hd + q * hd * d
    if shape.n_experts:
        touched = shape.n_experts * (1.0 - (1.0 - shape.top_k / shape.n_experts) ** rows)
        ffn, ffn_row = touched * 3 * d * shape.d_ff_expert + d * shape.n_experts, shape.top_k * 3 * d * shape.d_ff_expert + d * shape.n_experts
    else:
        ffn = ffn_row = 3 * d * shape.d_ff
    L, V = shape.n_layers, shape.vocab
    lm = d * V if logit_rows else 0
    visible, cached = keys
    return (2.0 * (L * (attn + ffn) + lm) + 2.0 * rows * d + 2.0 * 2 * L * kv * hd * (cached + rows) + 4.0 * logit_rows * V,
            2.0 * rows * L * (attn + ffn_row) + 2.0 * lm * logit_rows + 4.0 * L * q * hd * visible)


def work(case):
    t, d = _shapes(case)
    lens, B = _lens(case), case["batch"]
    passes = []
    if case["kind"] != "decode":
        for shape, ns in ((t, [n - 1 for n in lens]), (d, lens)):
            passes.append(_pass_work(shape, sum(ns), (sum(n * (n + 1) / 2 for n in ns), 0), 0))
    for it in range(case.get("iters", 0)):
        k, kt = case["k"], case["k"] + case["bonus"]
        at = [n + it for n in lens]   # a random block is hardly ever accepted at T = 0: one token per iteration
        ingest = B if it else 0
        passes.append(_pass_work(d, B * k + ingest, (sum((n + k) * k for n in at) + ingest * sum(at) / B, sum(at)), B * k))
        passes.append(_pass_work(t, B * kt, (sum(n * kt + kt * (kt - 1) / 2 for n in at), sum(n - 1 for n in at)), B * kt))
    return {"bytes": sum(p[0] for p in passes), "flops": sum(p[1] for p in passes)}


def tolerance(case):
    """Against the 64-bit reference the logits are off by 3e-6 to 6e-4 (few keys to average over: the larger ones), once
    by 4e-3, and a prefill's caches by up to 1.5e-3: a K or V value that lies near the middle of two bf16 values goes
    either way, which moves the rows above it, and in a mixture a row changes an expert now and then."""
    return {"rel": 6e-3, "max": 0.25, "differ": 0.01}


# ------------------------------------------------------------------------------------------------------------------
# the same in 64 bits
# ------------------------------------------------------------------------------------------------------------------
class _Model:
    """The decoder in float64 over sequences with caches of their own.  K and V rows are rounded to bf16 when they are
    made: that is what the caches hold and what the pass that makes them attends to."""

    def __init__(self, case, seed, model):
        self.shape, self.seed, self.model = _shapes(case)[model], seed, model
        s, n = self.shape, _max_seq(case)
        self.kv = torch.zeros(2, s.n_layers, case["batch"], n, s.n_kv_heads, s.head_dim, dtype=torch.bfloat16, device="cuda")
        if case["kind"] == "decode":
            for l in range(s.n_layers):
                for b, rows in enumerate(_cache_rows(s, seed, model, l, _lens(case))):
                    for i in range(2):
                        self.kv[i, l, b, : len(rows[i])] = rows[i]

    def w(self, name, layer=-1):
        return _weights(self.shape, self.seed, self.model, name, layer)

    def norm(self, x):
        return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + self.shape.rms_eps)

    def rope(self, x, pos):
        half = self.shape.head_dim // 2
        theta = self.shape.rope_base ** (-2.0 * torch.arange(half, device="cuda", dtype=torch.float64) / self.shape.head_dim)
        a = (pos.double()[:, None] * theta)[:, None]
        x1, x2 = x[..., :half], x[..., half:]
        return torch.cat([x1 * a.cos() - x2 * a.sin(), x2 * a.cos() + x1 * a.sin()], -1)

    def attend(self, q, layer, b, limit):
        """q [rows][head][dim], limit [rows]: visible keys."""
        s, n = self.shape, int(limit.max())
        k, v = (self.kv[i, layer, b, :n].double().permute(1, 0, 2).contiguous() for i in range(2))   # [kv head][key][dim]
        out = torch.empty_like(q)
        g = s.n_q_heads // s.n_kv_heads
        step = max(1, (1 << 28) // (s.n_q_heads * n))
        for r in range(0, len(q), step):
            qq = q[r : r + step]
            z = torch.matmul(qq.view(-1, s.n_kv_heads, g, s.head_dim).permute(1, 2, 0, 3).reshape(s.n_kv_heads, -1, s.head_dim).contiguous(),
                             k.transpose(1, 2).contiguous()).view(s.n_kv_heads, g, -1, n) / math.sqrt(s.head_dim)
            z.masked_fill_(torch.arange(n, device="cuda") >= limit[r : r + step, None], -math.inf)
            o = torch.matmul(z.softmax(-1).view(s.n_kv_heads, -1, n), v)
            out[r : r + step] = o.view(s.n_kv_heads, g, -1, s.head_dim).permute(2, 0, 1, 3).reshape(-1, s.n_q_heads, s.head_dim)
        return out

    def ffn(self, x, layer):
        s = self.shape
        swiglu = lambda x, wg, wu, wd: (torch.nn.functional.silu(x @ wg.double()) * (x @ wu.double())) @ wd.double()  # noqa: E731
        wg, wu, wd = (self.w(n, layer) for n in ("wg", "wu", "wd"))
        if not s.n_experts:
            return swiglu(x, wg, wu, wd)
        p, e = (x @ self.w("router", layer).double()).softmax(-1).topk(s.top_k, -1)
        p = p / p.sum(-1, keepdim=True)
        y = torch.zeros_like(x)
        for i in range(s.n_experts):
            row, slot = (e == i).nonzero(as_tuple=True)
            if len(row):
                y.index_add_(0, row, swiglu(x[row], wg[i], wu[i], wd[i]) * p[row, slot, None])
        return y

    def forward(self, rows):
        """rows: per sequence (tokens, positions = cache slots, limits), all on the GPU.  Returns the last hidden rows."""
        s = self.shape
        tok, pos, _ = (torch.cat([r[i] for r in rows]) for i in range(3))
        cuts = np.cumsum([0] + [len(r[0]) for r in rows]).tolist()
        x = self.w("embed")[tok.long()].double()
        for l in range(s.n_layers):
            h = self.norm(x)
            q, k, v = ((h @ self.w(n, l).double()).view(len(x), -1, s.head_dim) for n in ("wq", "wk", "wv"))
            q, k = self.rope(q, pos), self.rope(k, pos)
            o = torch.empty_like(q)
            for b, (_, p, limit) in enumerate(rows):
                at = slice(cuts[b], cuts[b + 1])
                if len(p):
                    self.kv[0, l, b, p.long()] = k[at].to(torch.bfloat16)
                    self.kv[1, l, b, p.long()] = v[at].to(torch.bfloat16)
                    o[at] = self.attend(q[at], l, b, limit)
            x = x + o.reshape(len(x), -1) @ self.w("wo", l).double()
            x = x + self.ffn(self.norm(x), l)
        return [x[cuts[b] : cuts[b + 1]] for b in range(len(rows))]

    def logits(self, x):
        return self.norm(x) @ self.w("lm_head").double()

    def blocks(self):
        """The caches as the library lays them out (see deer_get_kv_layout), [K, V][layer][sequence][kv head][block]..."""
        s = self.shape
        i, l, b, n, h, d = self.kv.shape
        x = self.kv.permute(0, 1, 2, 4, 3, 5).reshape(i, l, b, h, n // 32, 32, d)
        lane = torch.arange(64, device="cuda")
        r, half = lane % 32, lane // 32
        key = 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3)
        e = torch.arange(8, device="cuda")
        f = torch.arange(d // 16, device="cuda")[:, None, None]
        kk = x[0][..., key[None, :, None].expand(d // 16, 64, 8), 16 * f + 8 * half[:, None] + e]
        vv = x[1][..., 16 * half[:, None] + 8 * (f % 2) + e, (32 * (f // 2) + r[:, None]).expand(d // 16, 64, 8)]
        return torch.stack([kk, vv])


def exact(case, seed):
    lens, B = _lens(case), case["batch"]
    target, drafter = _Model(case, seed, 0), _Model(case, seed, 1)
    prompts, blocks = _tokens(case, seed)
    dev = lambda v: torch.tensor(v, device="cuda", dtype=torch.int64)  # noqa: E731
    if case["kind"] != "decode":
        for model, cut in ((target, 1), (drafter, 0)):
            model.forward([(dev(p[: len(p) - cut].tolist()), torch.arange(len(p) - cut, device="cuda"),
                            torch.arange(1, len(p) - cut + 1, device="cuda")) for p in prompts])
        if case["kind"] == "prefill":
            return {"target_cache": target.blocks(), "drafter_cache": drafter.blocks()}
    k, kt, vocab = case["k"], case["k"] + case["bonus"], target.shape.vocab
    seqs, pending, new = list(lens), [int(p[-1]) for p in prompts], [[] for _ in range(B)]
    for it in range(case["iters"]):
        rows = []
        for b, j in enumerate(seqs):
            m = len(new[b])
            at = torch.arange(j - m, j + k, device="cuda")
            limit = torch.where(at < j, at + 1, j + k)
            rows.append((dev(new[b] + [vocab - 1] * k), at, limit))
        zd = torch.stack([drafter.logits(x[-k:]) for x in drafter.forward(rows)])
        rows = [(dev(([pending[b]] + blocks[it][b].tolist())[:kt]), torch.arange(j - 1, j - 1 + kt, device="cuda"),
                 torch.arange(j, j + kt, device="cuda")) for b, j in enumerate(seqs)]
        zt = torch.stack([target.logits(x) for x in target.forward(rows)])
        if it + 1 < case["iters"]:   # greedy: the cases with more than one iteration are at T = 0
            best = zt.argmax(-1).tolist()
            for b in range(B):
                a = next((i for i in range(k) if best[b][i] != blocks[it][b][i]), k)
                new[b] = blocks[it][b][:a].tolist() + best[b][a : a + 1 if a < k else kt]
                seqs[b] += len(new[b])
                pending[b] = new[b][-1]
    kv = target.blocks()
    return {"draft_logits": zd, "verify_logits": zt, "accepted": None, "committed": None,
            "new_cache_rows": [kv[:, :, b, :, _new_blocks(case, b)] for b in range(B)]}
