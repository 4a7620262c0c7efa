"""What the speed of this library is measured on: the calls a program that
decodes with Ripple-Pivot Search makes, over their range of sizes.

listed() names the cases, draw() makes more of the same ranges, prepare()
makes what the program holds before the call, run() is one pass through the
public entry points, work() the bytes and operations it cannot do without,
tolerance() how far another correct implementation may be off, and exact()
the same outputs in 64 bits from plain torch and numpy.

Kinds of case:
  forward   Model.forward: a denoising forward, alone or over a cached prefix
  packed    Model.forward_packed: a lookahead packed into one sequence
  step      RpsStep.launch: pivots, branches, lookahead forward, score, commit
  lm_head   vocab_entropy_topk: LM head and vocabulary statistics alone
  schedule  the scheduler calls of a step on statistics that are there already

The models are the 8B-class shape, whole (32 layers) in two cases and cut to
four layers in most, the two-layer fp32 parity shape, and generic shapes with
64-wide heads; weights are N(0, 0.02).  The outputs of bf16 models are the
floating statistics: token ids of neighbouring ranks exchange places within
the rounding of bf16, so ids are returned where the logits are exact enough
to fix them (fp32 models, the LM head alone, the scheduler).
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2608_11742_amd as P
from paper_2608_11742_amd._abi import KvCache, Probe

DEV = "cuda:0"
TOPK = 16


def _shape(d, heads, hd, ffn, vocab):
    return dict(d_model=d, n_heads=heads, head_dim=hd, d_ffn=ffn, vocab=vocab, mask_id=vocab - 1, rope_base=10000.0,
                rms_eps=1e-5)


SHAPES = {
    "8b": _shape(4096, 32, 128, 12288, 126464),      # the 8B-class diffusion LLM
    "tiny": _shape(256, 4, 64, 1024, 1024),          # the fp32 parity model
    "small": _shape(1024, 16, 64, 4096, 32000),      # generic, 64-wide heads
    "mid": _shape(2048, 32, 64, 5632, 32000),        # generic, 64-wide heads, FFN not a power of two
}


# ---------------------------------------------------------------- the cases

def _forward(**kw):
    return dict(dict(kind="forward", model="8b", dtype="bf16", layers=4, batch=1, seq=512, prefix=0, n_lm=32,
                     kv_out=False, scaled=True), **kw)


def _packed(**kw):
    return dict(dict(kind="packed", model="8b", dtype="bf16", layers=4, shared=512, block=32, start=256, branches=10,
                     prefix=0, n_lm=32), **kw)


def _step(**kw):
    return dict(dict(kind="step", model="8b", dtype="bf16", layers=4, seq=512, n_m=256, prefix=0, pivots=4, cand=4),
                **kw)


def listed():
    return [
        # the scheduler's own calls between two forwards: 256 masked positions, 16 branches
        dict(kind="schedule", name="schedule_256", n_m=256, seq=512, pivots=4, cand=4),
        # the smallest whole step: 64 positions, two fp32 layers, 8 branches; launches and latency
        _step(name="step_tiny_f32", model="tiny", dtype="f32", layers=2, seq=64, n_m=32, pivots=2, cand=4),
        # an fp32 forward of ragged size
        _forward(name="forward_f32_3x201", model="small", dtype="f32", layers=4, batch=3, seq=201, n_lm=77),
        # the LM head alone on the masked rows of two blocks, an odd count
        dict(kind="lm_head", name="lm_head_61", rows=61, d=4096, vocab=126464, dtype="bf16"),
        # the later forwards of a decode over the prefix cache: the last block alone, batch 1
        _forward(name="block_1x32_over_1024", seq=32, prefix=1024, n_lm=32),
        # the same in the middle of a decode: block and masked suffix, some of the block committed
        _forward(name="suffix_1x160_over_352", seq=160, prefix=352, n_lm=17),
        # the forward that opens a block and fills the prefix cache
        _forward(name="open_1x512_kv", kv_out=True),
        # Algorithm 1's packed lookahead: anchor and ten candidates of one pivot
        _packed(name="packed_512_10x32"),
        # one RPS step over the prefix cache: 16 branches of a 32-position block
        _step(name="step_16x32_over_1024", seq=32, n_m=32, prefix=1024),
        # a batch of sequences of odd length through another model shape
        _forward(name="forward_mid_5x203", model="mid", layers=8, batch=5, seq=203, n_lm=101),
        # the whole 8B-class model: one denoising forward of 256 prompt and 256 masked positions
        _forward(name="forward_8b_1x512", layers=32, n_lm=256, scaled=False),
        # the whole 8B-class model: one lookahead step over 16 branches, the headline workload
        _step(name="step_8b_16x512", layers=32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "packed", "step", "lm_head", "schedule"])
    if kind == "schedule":
        n_m = _log(rng, 8, 1000)
        return dict(kind=kind, n_m=n_m, seq=n_m + _log(rng, 1, 1000), pivots=rng.randint(1, 4), cand=rng.randint(2, 4))
    if kind == "lm_head":
        d, vocab = rng.choice([(4096, 126464), (4096, 32000), (1024, 32000), (1024, 50257)])
        return dict(kind=kind, rows=_log(rng, 1, 4096), d=d, vocab=vocab, dtype="f32" if d == 1024 else "bf16")
    if kind == "packed":
        block = rng.choice([16, 32, 64])
        prefix = rng.choice([0, 0, _log(rng, 32, 1024)])
        blocks = rng.randint(1, 16)
        start = 0 if prefix else block * rng.randint(0, blocks - 1)
        return _packed(layers=rng.choice([2, 4]), shared=block * blocks, block=block, start=start,
                       branches=rng.randint(2, 15), prefix=prefix, n_lm=rng.randint(2, block))
    model = rng.choice(["8b", "8b", "8b", "mid", "small", "tiny"])
    dtype = {"8b": "bf16", "mid": "bf16", "small": rng.choice(["f32", "bf16"]), "tiny": "f32"}[model]
    layers = rng.choice([2, 4]) if model != "tiny" else 2
    if kind == "step":
        pivots, cand = rng.randint(1, 4), rng.randint(2, 4)
        prefix = rng.choice([0, _log(rng, 64, 2048)])
        n_m = rng.randint(8, 64) if prefix else rng.randint(16, 256)
        seq = n_m if prefix else n_m + rng.randint(1, 256)
        return _step(model=model, dtype=dtype, layers=layers, seq=seq, n_m=n_m, prefix=prefix, pivots=pivots, cand=cand)
    batch = rng.choice([1, 1, 1, rng.randint(2, 16)])
    seq = _log(rng, 8, 1024 if batch == 1 else 512)
    prefix = rng.choice([0, _log(rng, 32, 2048)])
    return _forward(model=model, dtype=dtype, layers=layers, batch=batch, seq=seq, prefix=prefix,
                    n_lm=rng.randint(1, seq), kv_out=batch == 1 and prefix == 0 and rng.random() < 0.5,
                    scaled=rng.random() < 0.5)


# ---------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _normal(gen, shape, std, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=gen)


def _weights(case, gen):
    s = SHAPES[case["model"]]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    d, f, v = s["d_model"], s["d_ffn"], s["vocab"]
    w = {"emb": _normal(gen, (v, d), 0.02, dt), "lm_head": _normal(gen, (v, d), 0.02, dt)}
    for l in range(case["layers"]):
        for name, shape in (("wqkv", (3 * d, d)), ("wo", (d, d)), ("wgu", (2 * f, d)), ("wdown", (d, f))):
            w[f"layers.{l}.{name}"] = _normal(gen, shape, 0.02, dt)
    return w


def _prefix(case, gen):
    """Keys and values of a cached prefix, with the spread the projections give."""
    if not case.get("prefix"):
        return None
    s, n, cap = SHAPES[case["model"]], case["prefix"], (case["prefix"] + 7) // 8 * 8
    bf = case["dtype"] == "bf16"
    std = 0.02 * math.sqrt(s["d_model"])
    k = _normal(gen, (case["layers"], s["n_heads"], cap, s["head_dim"]), std, torch.bfloat16 if bf else torch.float32)
    vt = _normal(gen, (case["layers"], s["n_heads"], s["head_dim"], cap), std,
                 torch.float16 if bf else torch.float32)
    return SimpleNamespace(k=k, vt=vt, n=n, cap=cap)


def _ints(gen, lo, hi, shape):
    return torch.randint(lo, hi, shape, generator=gen, device=DEV, dtype=torch.int32)


def _some(gen, n, of):
    """n of the numbers 0 .. of-1, ascending."""
    return torch.randperm(of, generator=gen, device=DEV)[:n].sort().values.to(torch.int32)


def _host_inputs(case, seed):
    """The inputs of a case as tensors: what prepare() hands to the library and exact() to its own arithmetic."""
    g = _gen(seed)
    h = SimpleNamespace()
    if case["kind"] == "lm_head":
        dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        h.hidden = _normal(g, (case["rows"], case["d"]), 1.0, dt)
        h.w = _normal(g, (case["vocab"], case["d"]), 0.02, dt)
        h.row_scale = torch.rand(case["rows"], generator=g, device=DEV) * 3.0 + 1.0
        return h
    if case["kind"] == "schedule":
        _carried(h, case, g, 32000, spread=(0.5, 6.0))
        n = case["pivots"] * case["cand"]
        h.branch = _statistics(g, n * case["n_m"], 32000, (0.3, 5.5))
        return h
    s = SHAPES[case["model"]]
    h.w = _weights(case, g)
    h.prefix = _prefix(case, g)
    if case["kind"] == "step":
        # entropies of unscaled logits lie near log(vocab) - 0.8; the carried ones a little above
        top = math.log(s["vocab"] - 1)
        _carried(h, case, g, s["vocab"], spread=(top - 0.75, top - 0.05))
        return h
    seq = case["seq"] if case["kind"] == "forward" else case["shared"]
    if case["kind"] == "forward":
        h.tokens = _ints(g, 0, s["vocab"] - 1, (case["batch"], seq))
        h.lm_pos = _some(g, case["n_lm"], seq)
        h.tokens[:, h.lm_pos.long()] = s["mask_id"]
    else:
        b0, B, nb = case["start"], case["block"], case["branches"]
        h.lm_pos = b0 + _some(g, case["n_lm"], B)
        shared = _ints(g, 0, s["vocab"] - 1, (seq,))
        shared[h.lm_pos.long()] = s["mask_id"]
        copies = shared[b0:b0 + B].repeat(nb, 1)
        h.probe_row = torch.full((nb,), int(case["n_lm"] // 2), dtype=torch.int32, device=DEV)
        h.probe_token = _ints(g, 0, s["vocab"] - 1, (nb,))
        copies[:, h.lm_pos[case["n_lm"] // 2].long() - b0] = h.probe_token
        h.tokens = torch.cat([shared, copies.reshape(-1)])
    h.row_scale = (1.0 + 3.0 * torch.rand(seq, generator=g, device=DEV)) if case.get("scaled", True) else None
    return h


def _statistics(gen, rows, vocab, spread):
    """Statistics of `rows` positions as a forward leaves them: distinct ids, descending logits."""
    gaps = torch.rand(rows, TOPK, generator=gen, device=DEV) * 0.3 + 0.05
    logit = 8.0 - gaps.cumsum(1)
    first = _ints(gen, 0, vocab - 1, (rows, 1))
    step = torch.arange(TOPK, device=DEV, dtype=torch.int32) * 997
    ids = (first + step) % (vocab - 1)
    lse = torch.logsumexp(logit, 1) + 0.2 + 2.0 * torch.rand(rows, generator=gen, device=DEV)
    H = spread[0] + (spread[1] - spread[0]) * torch.rand(rows, generator=gen, device=DEV)
    return SimpleNamespace(f3=torch.stack([H, lse, logit[:, 0]]), argmax=ids[:, 0].contiguous(), ids=ids.contiguous(),
                           logit=logit.contiguous())


def _carried(h, case, gen, vocab, spread):
    """One sequence whose last n_m positions are masked, and their carried statistics."""
    n, seq = case["n_m"], case["seq"]
    h.tokens = _ints(gen, 0, vocab - 1, (seq,))
    h.tokens[seq - n:] = vocab - 1
    h.m_pos = torch.arange(seq - n, seq, dtype=torch.int32, device=DEV)
    h.base = _statistics(gen, n, vocab, spread)


def _out_stats(R):
    """Stats whose three per-row floats share one [3][R] tensor."""
    st = P.Stats(R, TOPK, device=DEV)
    f3 = torch.zeros(3, R, dtype=torch.float32, device=DEV)
    st.H, st.lse, st.lmax = f3[0], f3[1], f3[2]
    return st, f3


def _load(st, f3, src):
    f3.copy_(src.f3)
    st.argmax.copy_(src.argmax)
    st.topk_id.copy_(src.ids)
    st.topk_logit.copy_(src.logit)


class _Restart:
    """The sequence, its masked positions and their carried statistics in one
    allocation, so that a step is started again from them with one copy."""

    def __init__(self, h, n, seq):
        words = seq + n + 4 * n + 2 * TOPK * n
        self.live = torch.empty(words, dtype=torch.int32, device=DEV)
        at = 0

        def take(count, shape, dtype=torch.int32):
            nonlocal at
            v = self.live[at:at + count].view(dtype).view(shape)
            at += count
            return v
        st = P.Stats(1, TOPK, device=DEV)
        self.f3 = take(3 * n, (3, n), torch.float32)
        st.H, st.lse, st.lmax = self.f3[0], self.f3[1], self.f3[2]
        st.topk_logit = take(TOPK * n, (n, TOPK), torch.float32)
        st.topk_id = take(TOPK * n, (n, TOPK))
        st.argmax = take(n, (n,))
        self.m_pos = take(n, (n,))
        self.tokens = take(seq, (seq,))
        self.base = st
        _load(st, self.f3, h.base)
        self.m_pos.copy_(h.m_pos)
        self.tokens.copy_(h.tokens)
        self.saved = self.live.clone()

    def restart(self):
        self.live.copy_(self.saved)


def _params(case):
    return P.params(mode="band", k_max=10, n_pivots=case["pivots"], r=0.0, n_cand=case["cand"],
                    max_branch=case["pivots"] * case["cand"])


LAMBDA = 0.1   # the decode's weight of a candidate's own probability


def prepare(case, seed):
    h = _host_inputs(case, seed)
    st = SimpleNamespace(case=case, kind=case["kind"])
    if st.kind == "lm_head":
        st.hidden, st.w, st.row_scale = h.hidden, h.w, h.row_scale
        st.out, st.f3 = _out_stats(case["rows"])
        st.ws = torch.empty(P.vocab_entropy_topk_workspace_bytes(case["rows"], case["vocab"]), dtype=torch.uint8,
                            device=DEV)
        return st
    if st.kind == "schedule":
        n, nb = case["n_m"], case["pivots"] * case["cand"]
        st.at = _Restart(h, n, case["seq"])
        st.prm, st.plan, st.dec = _params(case), P.new_plan(DEV), P.new_decision(DEV)
        st.branch, f3 = _out_stats(nb * n)
        _load(st.branch, f3, h.branch)
        st.branch_tokens = torch.empty(nb, case["seq"], dtype=torch.int32, device=DEV)
        st.scores, st.deltas = torch.zeros(16, device=DEV), torch.zeros(16, device=DEV)
        st.n_m_out = torch.zeros(1, dtype=torch.int32, device=DEV)
        st.committed = torch.zeros(n, dtype=torch.int32, device=DEV)
        st.n_committed = torch.zeros(1, dtype=torch.int32, device=DEV)
        return st
    shape = SimpleNamespace(n_layers=case["layers"], **SHAPES[case["model"]])
    seq = {"forward": "seq", "step": "seq", "packed": "shared"}[st.kind]
    st.model = P.Model(shape, h.w, dtype=case["dtype"], max_pos=case["prefix"] + case[seq])
    st.kv = None
    if h.prefix is not None:
        st.prefix = h.prefix
        st.kv = KvCache(h.prefix.k.data_ptr(), h.prefix.vt.data_ptr(), h.prefix.n, h.prefix.cap)
    if st.kind == "step":
        st.at = _Restart(h, case["n_m"], case["seq"])
        st.step = P.RpsStep(st.model, st.at.tokens, st.at.m_pos, st.at.base, _params(case), lam=LAMBDA,
                            capacity=case["pivots"] * case["cand"], kv_prefix=st.kv, pos_offset=case["prefix"])
        R = st.step.branch_stats.R
        st.step.branch_stats, st.f3 = _out_stats(R)
        return st
    st.tokens, st.lm_pos, st.row_scale = h.tokens, h.lm_pos, h.row_scale
    if st.kind == "packed":
        st.out, st.f3 = _out_stats((1 + case["branches"]) * case["n_lm"])
        st.probe_row, st.probe_token = h.probe_row, h.probe_token
        st.probe_logit = torch.zeros(case["branches"], device=DEV)
        st.probe = Probe(st.probe_row.data_ptr(), st.probe_token.data_ptr(), st.probe_logit.data_ptr(),
                         case["branches"])
        st.model.workspace_packed(case["shared"], case["block"], case["branches"], case["n_lm"])
        return st
    st.out, st.f3 = _out_stats(case["batch"] * case["n_lm"])
    st.kv_out = None
    if case["kv_out"]:
        k, vt, cap = st.model.new_kv_cache(case["seq"])
        st.cache = (k.zero_(), vt.zero_())
        st.kv_out = KvCache(k.data_ptr(), vt.data_ptr(), 0, cap)
    st.model.workspace(case["batch"], case["seq"], case["n_lm"])
    return st


# ---------------------------------------------------------------- one pass

def run(st):
    case = st.case
    if st.kind == "lm_head":
        P.vocab_entropy_topk(st.hidden, st.w, st.out, st.ws, row_scale=st.row_scale, mask_id=case["vocab"] - 1)
        return {"rows": st.f3, "topk_logit": st.out.topk_logit, "argmax": st.out.argmax, "topk_id": st.out.topk_id}
    if st.kind == "schedule":
        a, n, nb = st.at, case["n_m"], case["pivots"] * case["cand"]
        a.restart()
        P.rps_select_pivots(a.base, a.m_pos, n, st.prm, st.plan)
        P.rps_build_branches(a.tokens, st.plan, False, nb, st.branch_tokens)
        P.rps_lookahead_score(a.base, st.branch, 0, n, st.plan, LAMBDA, st.dec, scores=st.scores, deltas=st.deltas)
        P.rps_commit(a.tokens, a.m_pos, n, a.base, 0.3, st.n_m_out, st.committed, st.n_committed, dec=st.dec,
                     branches=st.branch, branch_offset=0)
        return {"tokens": a.tokens, "m_pos": a.m_pos, "rows": a.f3, "topk_logit": a.base.topk_logit,
                "topk_id": a.base.topk_id, "argmax": a.base.argmax, "scores": st.scores, "deltas": st.deltas,
                "branch_tokens": st.branch_tokens, "n_m": st.n_m_out, "committed": st.committed,
                "n_committed": st.n_committed}
    if st.kind == "step":
        s = st.step
        st.at.restart()
        s.launch()
        out = {"branch_rows": st.f3, "branch_topk_logit": s.branch_stats.topk_logit, "branch_tokens": s.branch_tokens,
               "scores": s.scores, "tokens": st.at.tokens, "m_pos": st.at.m_pos, "rows": st.at.f3,
               "topk_logit": st.at.base.topk_logit, "n_m": s.n_m_out, "n_committed": s.n_committed}
        if case["dtype"] == "f32":
            out["branch_topk_id"] = s.branch_stats.topk_id
        return out
    if st.kind == "packed":
        st.model.forward_packed(st.tokens, case["shared"], case["start"], case["block"], case["branches"], st.lm_pos,
                                out=st.out, row_scale=st.row_scale, pos_offset=case["prefix"], kv_prefix=st.kv,
                                probe=st.probe)
        # the probed logits are left out: those of arbitrary tokens lie around zero, within a few times bf16's rounding
        return {"rows": st.f3, "topk_logit": st.out.topk_logit}
    st.model.forward(st.tokens, st.lm_pos, out=st.out, row_scale=st.row_scale, pos_offset=case["prefix"],
                     kv_prefix=st.kv, kv_out=st.kv_out)
    out = {"rows": st.f3, "topk_logit": st.out.topk_logit}
    if case["dtype"] == "f32":
        out["topk_id"] = st.out.topk_id
    if st.kv_out is not None:
        out["cache_k"], out["cache_v"] = st.cache
    return out


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    if case["kind"] == "schedule":
        n, nb = case["n_m"], case["pivots"] * case["cand"]
        row = (4 + 2 * TOPK) * 4
        # the carried rows and the winner's, read once; carried rows and branch sequences written once
        return {"bytes": n * row * 3 + nb * n * 4 + nb * case["seq"] * 4 + 2 * case["seq"] * 4,
                "flops": n * 40 + nb * n * 2}
    T = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "lm_head":
        R, d, v = case["rows"], case["d"], case["vocab"]
        return {"bytes": (R * d + v * d) * T + R * (4 + 2 * TOPK) * 4, "flops": 2 * R * d * v}
    s, L = SHAPES[case["model"]], case["layers"]
    d, f, v = s["d_model"], s["d_ffn"], s["vocab"]
    if case["kind"] == "packed":
        rows = case["shared"] + case["branches"] * case["block"]
        keys = case["shared"] + case["prefix"]
        R = (1 + case["branches"]) * case["n_lm"]
    else:
        batch = case["batch"] if case["kind"] == "forward" else case["pivots"] * case["cand"]
        rows, keys = batch * case["seq"], case["seq"] + case["prefix"]
        R = batch * (case["n_lm"] if case["kind"] == "forward" else case["n_m"])
    weights = L * (4 * d * d + 3 * d * f) + v * d
    flops = L * (2 * rows * (4 * d * d + 3 * d * f) + 4 * rows * keys * d) + 2 * R * d * v
    kv = 2 * L * case["prefix"] * d * T + (2 * L * rows * d * T if case.get("kv_out") else 0)
    return {"bytes": weights * T + rows * (4 + d * T) + kv + R * (4 + 2 * TOPK) * 4, "flops": flops}


def tolerance(case):
    """About four times what 16-bit storage of activations, keys and values
    (or the order of 32-bit sums) moved the outputs by against exact() on an
    MI355X: bf16 statistics and top logits 0.2 to 0.35 %, cached keys and
    values 0.9 %, fp32 models 6e-7, the LM head alone 4e-7, scores 9e-8."""
    if case["kind"] == "schedule":
        return {"rel": 1e-6, "max": 1e-4}
    if case["kind"] == "lm_head" or case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 2e-4, "differ": 0.01}
    if case.get("kv_out"):
        return {"rel": 3e-2, "max": 0.8}
    return {"rel": 1.4e-2, "max": 0.3}


# ---------------------------------------------------------------- the same in 64 bits

def _ref_layers(case, h, tokens, pos, mask):
    """Final normed hidden states [B][S][d] in float64, and every layer's K and V [B][H][S][hd].
    tokens [B][S], pos [S] position ids, mask None or [S][S] (True: visible)."""
    s = SHAPES[case["model"]]
    H, hd = s["n_heads"], s["head_dim"]
    B, S = tokens.shape
    x = h.w["emb"][tokens.long()].double()

    def norm(t):
        return t / torch.sqrt(t.square().mean(-1, keepdim=True) + s["rms_eps"])

    inv = s["rope_base"] ** (-2.0 * torch.arange(hd // 2, device=DEV, dtype=torch.float64) / hd)
    ang = pos.double()[:, None] * inv[None]
    cos, sin = ang.cos(), ang.sin()

    def rope(t):
        a, b = t[..., :hd // 2], t[..., hd // 2:]
        return torch.cat([a * cos - b * sin, a * sin + b * cos], -1)

    kv = []
    for l in range(case["layers"]):
        w = {n: h.w[f"layers.{l}.{n}"].double() for n in ("wqkv", "wo", "wgu", "wdown")}
        qkv = (norm(x).view(B * S, -1) @ w["wqkv"].T).view(B, S, 3, H, hd).permute(2, 0, 3, 1, 4)
        q, k, v = rope(qkv[0]), rope(qkv[1]), qkv[2]
        kv.append((k, v))
        o = torch.empty(B, S, H, hd, dtype=torch.float64, device=DEV)
        for b in range(B):
            sc = torch.bmm(q[b].contiguous(), k[b].transpose(1, 2).contiguous()) / math.sqrt(hd)
            if mask is not None:
                sc = sc.masked_fill(~mask, -math.inf)
            vb = v[b]
            if h.prefix is not None:
                n = h.prefix.n
                pk, pv = h.prefix.k[l, :, :n].double(), h.prefix.vt[l, :, :, :n].double().transpose(1, 2)
                sc = torch.cat([torch.bmm(q[b].contiguous(), pk.transpose(1, 2).contiguous()) / math.sqrt(hd), sc], 2)
                vb = torch.cat([pv, vb], 1)
            o[b] = torch.bmm(sc.softmax(-1), vb.contiguous()).transpose(0, 1)
        x = x + (o.view(B * S, -1) @ w["wo"].T).view(B, S, -1)
        gu = norm(x).view(B * S, -1) @ w["wgu"].T
        f = gu.shape[1] // 2
        act = torch.nn.functional.silu(gu[:, :f]) * gu[:, f:]
        x = x + (act @ w["wdown"].T).view(B, S, -1)
    return norm(x), kv


def _ref_stats(hidden, w_lm, scale, mask_id):
    """hidden [R][d] float64, scale [R] or None: [3][R] (H, lse, lmax), top-k ids and logits."""
    wd = w_lm.double()
    rows, ids, vals = [], [], []
    for r in range(0, hidden.shape[0], 256):
        lg = hidden[r:r + 256] @ wd.T
        if scale is not None:
            lg = lg * scale[r:r + 256, None].double()
        lg[:, mask_id] = -math.inf
        lse = torch.logsumexp(lg, 1)
        p = (lg - lse[:, None]).exp()
        ent = lse - (p * lg.nan_to_num(neginf=0.0)).sum(1)
        v, i = lg.topk(TOPK, 1)
        rows.append(torch.stack([ent, lse, v[:, 0]]))
        ids.append(i)
        vals.append(v)
    return torch.cat(rows, 1), torch.cat(ids).to(torch.int32), torch.cat(vals)


def _ref_plan(h, case):
    """Band-mode pivots and their candidates, in plan order: [(row, position, token, log p)]."""
    f3 = h.base.f3.double().cpu().numpy()
    logit, ids = h.base.logit.double().cpu().numpy(), h.base.ids.cpu().numpy()
    ent, lse = f3[0], f3[1]
    lo, hi = np.percentile(ent, 25.0), np.percentile(ent, 75.0)
    lp = logit[:, :10] - lse[:, None]
    ht = -(np.exp(lp) * lp).sum(1)
    rows = sorted((j for j in range(len(ent)) if lo <= ent[j] <= hi), key=lambda j: (-ht[j], j))[:case["pivots"]]
    first = case["seq"] - case["n_m"]
    return [(j, first + j, int(ids[j, c]), float(lp[j, c])) for j in rows for c in range(case["cand"])]


def _ref_branches(h, case, plan):
    t = h.tokens.repeat(case["pivots"] * case["cand"], 1)
    for b, (_, pos, token, _) in enumerate(plan):
        t[b, pos] = token
    return t


def _ref_scores(h, plan, branch_H):
    """Eq. 4 of each branch and its margin over the pivot's [MASK] score; branch_H [branches][n_m]."""
    f3 = h.base.f3.double().cpu().numpy()
    bh = branch_H.double().cpu().numpy()
    n = bh.shape[1]
    scores, deltas = np.zeros(16), np.zeros(16)
    for b, (row, _, _, lp) in enumerate(plan):
        keep = np.arange(n) != row
        scores[b] = -bh[b][keep].sum() / (n - 1) + LAMBDA * lp
        deltas[b] = (f3[0] - bh[b])[keep].sum() / (n - 1) + LAMBDA * (lp - (f3[2, row] - f3[1, row]))
    return torch.from_numpy(scores), torch.from_numpy(deltas)


def exact(case, seed):
    h = _host_inputs(case, seed)
    if case["kind"] == "lm_head":
        rows, ids, vals = _ref_stats(h.hidden.double(), h.w, h.row_scale, case["vocab"] - 1)
        return {"rows": rows, "topk_logit": vals, "argmax": ids[:, 0], "topk_id": ids}
    if case["kind"] == "schedule":
        plan = _ref_plan(h, case)
        nb = len(plan)
        scores, deltas = _ref_scores(h, plan, h.branch.f3[0].view(-1, case["n_m"])[:nb])
        return {"tokens": None, "m_pos": None, "rows": None, "topk_logit": None, "topk_id": None, "argmax": None,
                "scores": scores, "deltas": deltas, "branch_tokens": _ref_branches(h, case, plan), "n_m": None,
                "committed": None, "n_committed": None}
    s, base = SHAPES[case["model"]], case["prefix"]
    if case["kind"] == "packed":
        S, b0, B, nb = case["shared"], case["start"], case["block"], case["branches"]
        n = S + nb * B
        pos = torch.cat([torch.arange(S, device=DEV), torch.arange(b0, b0 + B, device=DEV).repeat(nb)]) + base
        mask = torch.zeros(n, n, dtype=torch.bool, device=DEV)
        mask[:, :S] = True
        mask[S:, b0:b0 + B] = False
        for j in range(nb):
            mask[S + j * B:S + (j + 1) * B, S + j * B:S + (j + 1) * B] = True
        hid, _ = _ref_layers(case, h, h.tokens[None], pos, mask)
        lm = h.lm_pos.long()
        at = torch.cat([lm] + [S + j * B + (lm - b0) for j in range(nb)])
        scale = h.row_scale[lm].repeat(1 + nb)
        hid = hid[0, at]
        rows, _, vals = _ref_stats(hid, h.w["lm_head"], scale, s["mask_id"])
        return {"rows": rows, "topk_logit": vals}
    if case["kind"] == "step":
        plan = _ref_plan(h, case)
        tokens = _ref_branches(h, case, plan)
        hid, _ = _ref_layers(case, h, tokens, torch.arange(case["seq"], device=DEV) + base, None)
        hid = hid[:, case["seq"] - case["n_m"]:].reshape(-1, s["d_model"])
        rows, ids, vals = _ref_stats(hid, h.w["lm_head"], None, s["mask_id"])
        scores, _ = _ref_scores(h, plan, rows[0].view(-1, case["n_m"]))
        out = {"branch_rows": rows, "branch_topk_logit": vals, "branch_tokens": tokens, "scores": scores,
               "tokens": None, "m_pos": None, "rows": None, "topk_logit": None, "n_m": None, "n_committed": None}
        if case["dtype"] == "f32":
            out["branch_topk_id"] = ids
        return out
    hid, kv = _ref_layers(case, h, h.tokens, torch.arange(case["seq"], device=DEV) + base, None)
    hid = hid[:, h.lm_pos.long()].reshape(-1, s["d_model"])
    scale = h.row_scale[h.lm_pos.long()].repeat(case["batch"]) if h.row_scale is not None else None
    rows, ids, vals = _ref_stats(hid, h.w["lm_head"], scale, s["mask_id"])
    out = {"rows": rows, "topk_logit": vals}
    if case["dtype"] == "f32":
        out["topk_id"] = ids
    if case["kv_out"]:
        cap = (case["seq"] + 7) // 8 * 8
        k = torch.zeros(case["layers"], s["n_heads"], cap, s["head_dim"], dtype=torch.float64, device=DEV)
        v = torch.zeros(case["layers"], s["n_heads"], s["head_dim"], cap, dtype=torch.float64, device=DEV)
        for l, (kl, vl) in enumerate(kv):
            k[l, :, :case["seq"]] = kl[0]
            v[l, :, :, :case["seq"]] = vl[0].transpose(1, 2)
        out["cache_k"], out["cache_v"] = k, v
    return out
