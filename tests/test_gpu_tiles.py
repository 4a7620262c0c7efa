"""GPU parity where a tile or a split begins, ends or is left partly filled:
one small forward per edge against the CPU oracle."""
import numpy as np
import pytest
import torch

import synth
from synth import ModelShape
from oracle import model as om
from oracle.stats import softmax_stats
from tests.parity import compare_stats

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def P():
    import paper_2608_11742_amd as P
    return P


# fp32: 64 x 64 projection tiles of one head (hd 64) or half a head (hd 128),
# split and unsplit K; rows one below, at and one above a row tile, a batch
# whose sequences straddle tiles, and an FFN whose half tiles end unevenly
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("B_,S", [(1, 1), (1, 63), (1, 64), (1, 65), (3, 43), (2, 320)])
def test_forward_f32_row_tiles(P, hd, B_, S):
    shape = ModelShape(n_layers=2, d_model=512, n_heads=512 // hd, head_dim=hd, d_ffn=640, vocab=700)
    w_np = synth.model_weights_np(shape, seed=3, dtype="f32")
    model = P.Model(shape, {k: torch.from_numpy(v).to(DEV) for k, v in w_np.items()}, dtype="f32", max_pos=512)
    toks = synth.tokens_np(7, "toks", B_ * S, shape.vocab - 1).reshape(B_, S)
    toks[:, S // 2:] = shape.mask_id
    lm_pos = np.unique(np.array([0, S // 3, S // 2, S - 1], dtype=np.int32))
    out = model.forward(torch.from_numpy(toks).to(DEV), torch.from_numpy(lm_pos).to(DEV), scale=2.0)
    torch.cuda.synchronize()
    ref = softmax_stats(om.forward_logits(toks, w_np, shape, lm_pos, scale=2.0).reshape(-1, shape.vocab), 16)
    print(compare_stats(out.numpy(), ref, 1e-4, label=f"f32 hd {hd} {B_} x {S}"))
    model.close()


# LM head: 64-, 128- and 256-row tiles, rows and vocabularies around a tile
# edge, one slice and many, the merge of 1 to 8 waves of partials
@pytest.mark.parametrize("dtype,R,d,V", [
    ("bf16", 64, 128, 127), ("bf16", 65, 128, 129), ("bf16", 3, 64, 33000), ("bf16", 130, 64, 40000),
    ("f32", 64, 64, 1024), ("f32", 65, 64, 33000), ("f32", 300, 32, 2049), ("f32", 33000, 32, 260)])
def test_lm_head_tiles(P, dtype, R, d, V):
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    h = synth.hidden_np(11, "h", (R, d), dtype=dtype)
    w = synth.weight_np(12, "w", (V, d), std=0.1, dtype=dtype)
    mask = V // 2
    out = P.Stats(R, 16, device=DEV).fill_(float("nan"))
    ws = torch.full((P.vocab_entropy_topk_workspace_bytes(R, V),), 255, dtype=torch.uint8, device=DEV)
    P.vocab_entropy_topk(torch.from_numpy(h).to(DEV).to(td), torch.from_numpy(w).to(DEV).to(td), out, ws, scale=2.0,
                         mask_id=mask)
    torch.cuda.synchronize()
    logits = 2.0 * (h.astype(np.float64) @ w.astype(np.float64).T)
    logits[:, mask] = -np.inf
    print(compare_stats(out.numpy(), softmax_stats(logits, 16), 1e-4 if dtype == "f32" else 1e-3,
                        label=f"lm head {dtype} {R} x {V}"))


@pytest.mark.parametrize("R,V,k", [(2, 40000, 16), (70, 33000, 5), (1, 12, 16)])
def test_lm_head_of_equal_logits(P, R, V, k):
    """Ties everywhere: the ids ascend, and the merge's bound, which breaks
    ties by id, keeps few of the lists.  With fewer tokens than ranks the rest
    stay empty."""
    out = P.Stats(R, k, device=DEV).fill_(float("nan"))
    ws = torch.empty(P.vocab_entropy_topk_workspace_bytes(R, V), dtype=torch.uint8, device=DEV)
    P.vocab_entropy_topk(torch.zeros(R, 64, dtype=torch.bfloat16, device=DEV),
                         torch.ones(V, 64, dtype=torch.bfloat16, device=DEV), out, ws, mask_id=3)
    got = out.numpy()
    want = [i for i in range(min(V, 17)) if i != 3][:k]
    assert (got["topk_id"][:, :len(want)] == want).all() and (got["topk_logit"][:, :len(want)] == 0).all()
    assert np.isneginf(got["topk_logit"][:, len(want):]).all()
    assert (got["argmax"] == 0).all() and np.allclose(got["H"], np.log(V - 1), atol=1e-4)


def test_lm_head_merge_of_more_candidates_than_its_buffer(P):
    """2048 partials of 32 tokens, thread t of the merge takes t, t + 512, ...
    Fifteen threads of its wave 0 and of its wave 4 see one high logit in every
    token they hold, the sixteenth of each a lower one, which is the bound:
    30 x 4 lists of 16 reach it, 1920 candidates and more for a buffer of 1024.
    The top 16 are spread over the lists."""
    V, n = 65536, 16
    part = np.arange(V) // 32 % 512
    val = np.zeros(V, np.float32)
    val[np.isin(part, np.r_[0:15, 256:271])] = 2.0
    val[part == 15], val[part == 271] = 1.0, 0.5
    top = np.array([(512 * (j % 4) + (j % 15) + 256 * (j % 2)) * 32 + 3 * j % 32 for j in range(n)])
    val[top] = 2.5 + 0.125 * np.arange(n)
    w = torch.zeros(V, 64, dtype=torch.bfloat16, device=DEV)
    w[:, 0] = torch.from_numpy(val).to(DEV)
    h = torch.zeros(2, 64, dtype=torch.bfloat16, device=DEV)
    h[0, 0], h[1, 0] = 1.0, 2.0
    out = P.Stats(2, 16, device=DEV).fill_(float("nan"))
    ws = torch.full((P.vocab_entropy_topk_workspace_bytes(2, V),), 255, dtype=torch.uint8, device=DEV)
    P.vocab_entropy_topk(h, w, out, ws)
    got = out.numpy()
    assert (got["topk_id"] == top[::-1]).all() and (got["argmax"] == top[-1]).all()
    print(compare_stats(got, softmax_stats(np.stack([val, 2 * val]).astype(np.float64), 16), 1e-4, label="merge"))


# scheduler: rows one below, at and one above the commit kernel's 256 threads
# and its limit of 1024, every kept row in order; positions past the sequence
# are clamped, the last row that lands on a token wins
@pytest.mark.parametrize("n_m", [1, 63, 64, 65, 255, 256, 257, 1000, 1024])
@pytest.mark.parametrize("shift", [0, 5])
def test_commit_rows(P, n_m, shift):
    rng = np.random.default_rng(n_m)
    seq, k = n_m + 7, 4
    base = P.Stats(n_m, k, device=DEV)
    f = {n: rng.normal(size=getattr(base, n).shape).astype(np.float32) for n in ("H", "lse", "lmax", "topk_logit")}
    f["lmax"] = f["lse"] - 1.0 - np.abs(f["lmax"])
    f["lmax"][rng.random(n_m) < 0.4] = f["lse"][0] = 0.0
    f["lse"][f["lmax"] == 0.0] = 0.05
    i = {n: rng.integers(0, 9000, getattr(base, n).shape).astype(np.int32) for n in ("argmax", "topk_id")}
    for n, v in {**f, **i}.items():
        getattr(base, n).copy_(torch.from_numpy(v))
    pos = np.arange(7 + shift, seq + shift, dtype=np.int32)
    tokens = rng.integers(0, 9000, seq).astype(np.int32)
    t, m = torch.from_numpy(tokens).to(DEV), torch.from_numpy(pos).to(DEV)
    one = lambda n: torch.full((n,), -7, dtype=torch.int32, device=DEV)
    n_out, com, n_com = one(1), one(n_m), one(1)
    P.rps_commit(t, m, n_m, base, 0.9, n_out, com, n_com)
    conf = np.exp((f["lmax"] - f["lse"]).astype(np.float64))
    sel = conf >= 0.9
    if not sel.any():
        sel[np.argmax(conf)] = True
    want = tokens.copy()
    for j in np.flatnonzero(sel):
        want[min(pos[j], seq - 1)] = i["argmax"][j]
    keep = ~sel
    assert n_out.item() == keep.sum() and n_com.item() == sel.sum()
    assert (com.cpu().numpy()[:sel.sum()] == pos[sel]).all() and (t.cpu().numpy() == want).all()
    assert (m.cpu().numpy()[:keep.sum()] == pos[keep]).all()
    got = base.numpy()
    for n, v in {**f, **i}.items():
        assert (got[n][:keep.sum()] == v[keep]).all(), n


# a decision to commit: its pivot's row goes, its token stands, and the rule and
# the rows that are kept are the winning branch's
@pytest.mark.parametrize("n_m", [2, 255, 256, 257, 1000, 1024])
@pytest.mark.parametrize("where", ["first", "middle", "last"])
def test_commit_of_a_pivot(P, n_m, where):
    from paper_2608_11742_amd._abi import RpsDecision
    rng = np.random.default_rng(n_m)
    seq, k, nb = n_m + 7, 4, 3
    row = {"first": 0, "middle": n_m // 2, "last": n_m - 1}[where]
    pos = np.arange(7, seq, dtype=np.int32)
    base, br = P.Stats(n_m, k, device=DEV).fill_(0.0), P.Stats((1 + nb) * n_m, k, device=DEV)
    f = {n: rng.normal(size=getattr(br, n).shape).astype(np.float32) for n in ("H", "lse", "lmax", "topk_logit")}
    sure = rng.random((1 + nb) * n_m) < 0.4
    f["lmax"] = f["lse"] - np.where(sure, np.float32(0.05), np.float32(1.0) + np.abs(f["lmax"]))
    i = {n: rng.integers(0, 9000, getattr(br, n).shape).astype(np.int32) for n in ("argmax", "topk_id")}
    for n, v in {**f, **i}.items():
        getattr(br, n).copy_(torch.from_numpy(v))
    branch, offset = 2, 1
    win = slice((offset + branch) * n_m, (offset + branch + 1) * n_m)
    dec = P.new_decision(DEV)
    dec.copy_(torch.frombuffer(bytearray(bytes(RpsDecision(1, branch, row, int(pos[row]), 8999, 0.5, 0.1, n_m))),
                               dtype=torch.uint8))
    tokens = rng.integers(0, 8000, seq).astype(np.int32)
    t, m = torch.from_numpy(tokens).to(DEV), torch.from_numpy(pos).to(DEV)
    one = lambda n: torch.full((n,), -7, dtype=torch.int32, device=DEV)
    n_out, com, n_com = one(1), one(n_m), one(1)
    P.rps_commit(t, m, n_m, base, 0.9, n_out, com, n_com, dec=dec, branches=br, branch_offset=offset)
    conf = np.exp((f["lmax"][win] - f["lse"][win]).astype(np.float64))
    conf[row] = -1.0
    sel = conf >= 0.9
    if not sel.any():
        sel[np.argmax(conf)] = True
    want = tokens.copy()
    want[pos[row]] = 8999
    want[pos[sel]] = i["argmax"][win][sel]
    keep = ~sel
    keep[row] = False
    n = keep.sum()
    assert n_out.item() == n and n_com.item() == 1 + sel.sum()
    assert (com.cpu().numpy()[:1 + sel.sum()] == np.concatenate([pos[row:row + 1], pos[sel]])).all()
    assert (t.cpu().numpy() == want).all() and (m.cpu().numpy()[:n] == pos[keep]).all()
    got = base.numpy()
    for name, v in {**f, **i}.items():
        assert (got[name][:n] == v[win][keep]).all(), name


def test_commit_without_any_confidence(P):
    """Statistics of a model gone to NaN: the first row commits, so that a decode ends."""
    base = P.Stats(70, 4, device=DEV).fill_(float("nan"))
    base.argmax.copy_(torch.arange(70, dtype=torch.int32))
    t, m = torch.zeros(80, dtype=torch.int32, device=DEV), torch.arange(5, 75, dtype=torch.int32, device=DEV)
    n_out, com, n_com = (torch.zeros(n, dtype=torch.int32, device=DEV) for n in (1, 70, 1))
    P.rps_commit(t, m, 70, base, 0.9, n_out, com, n_com)
    assert n_out.item() == 69 and n_com.item() == 1 and com[0].item() == 5
    assert (m[:69].cpu() == torch.arange(6, 75)).all()


@pytest.mark.parametrize("n_m", [2, 64, 300, 1024])
@pytest.mark.parametrize("order", ["pairs", "shuffled", "all"])
def test_commit_of_repeated_positions(P, n_m, order):
    """Several rows at one position: committed[] lists them all, and the last
    row's token stays, whichever waves the rows are in."""
    rng = np.random.default_rng(n_m)
    seq = n_m + 3
    pos = {"pairs": np.arange(n_m) // 2, "shuffled": rng.permutation(n_m) // 3, "all": np.full(n_m, 2)}[order]
    pos = pos.astype(np.int32)
    base = P.Stats(n_m, 4, device=DEV).fill_(0.0)
    ids = rng.permutation(9000)[:n_m].astype(np.int32)
    base.argmax.copy_(torch.from_numpy(ids))
    tokens = np.full(seq, -1, np.int32)
    t, m = torch.from_numpy(tokens).to(DEV), torch.from_numpy(pos).to(DEV)
    one = lambda n: torch.full((n,), -7, dtype=torch.int32, device=DEV)
    n_out, com, n_com = one(1), one(n_m), one(1)
    P.rps_commit(t, m, n_m, base, 0.5, n_out, com, n_com)
    for j in range(n_m):
        tokens[pos[j]] = ids[j]
    assert n_out.item() == 0 and n_com.item() == n_m
    assert (com.cpu().numpy() == pos).all() and (t.cpu().numpy() == tokens).all()


# bf16 projections: rows at the edges of the 64-, 128- and 256-row tiles and of
# the ranges that choose between them, an FFN whose last tile is partly filled
@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("B_,S", [(1, 33), (1, 64), (1, 65), (2, 64), (1, 129), (1, 300), (1, 513), (3, 500), (6, 500)])
def test_forward_bf16_row_tiles(P, hd, B_, S):
    shape = ModelShape(n_layers=1, d_model=1024, n_heads=1024 // hd, head_dim=hd, d_ffn=2816, vocab=600)
    w_np = synth.model_weights_np(shape, seed=4, dtype="bf16")
    model = P.Model(shape, {k: torch.from_numpy(v).to(DEV).bfloat16() for k, v in w_np.items()}, dtype="bf16",
                    max_pos=512 + 64)
    toks = synth.tokens_np(8, "toks", B_ * S, shape.vocab - 1).reshape(B_, S)
    toks[:, S // 2:] = shape.mask_id
    lm_pos = np.unique(np.array([0, 1, S // 3, S // 2, S - 2, S - 1], dtype=np.int32))
    out = model.forward(torch.from_numpy(toks).to(DEV), torch.from_numpy(lm_pos).to(DEV), scale=2.0)
    torch.cuda.synchronize()
    got, n = out.numpy(), len(lm_pos)
    for b in {0, B_ - 1}:
        ref = softmax_stats(om.forward_logits(toks[b:b + 1], w_np, shape, lm_pos, scale=2.0, mirror=True).reshape(
            -1, shape.vocab), 16)
        print(compare_stats({k: v[b * n:(b + 1) * n] for k, v in got.items()}, ref, 2e-2, max_exceptions=2,
                            id_ranks=4, label=f"bf16 hd {hd} {B_} x {S} seq {b}"))
    model.close()


# the smallest bf16 models: K too short for parts, so that up to 64 rows take
# every unsplit 64 x 128 kernel; 65-128 rows with a small FFN, whose gate/up
# runs in parts of 128 x 128 tiles
@pytest.mark.parametrize("d,hd,F,S", [(256, 64, 256, 1), (256, 64, 256, 33), (256, 64, 256, 64), (256, 128, 256, 1),
                                      (256, 128, 256, 33), (256, 128, 256, 64), (512, 64, 640, 65),
                                      (512, 128, 640, 128)])
def test_forward_bf16_small_models(P, d, hd, F, S):
    shape = ModelShape(n_layers=1, d_model=d, n_heads=d // hd, head_dim=hd, d_ffn=F, vocab=600)
    w_np = synth.model_weights_np(shape, seed=7, dtype="bf16")
    model = P.Model(shape, {k: torch.from_numpy(v).to(DEV).bfloat16() for k, v in w_np.items()}, dtype="bf16",
                    max_pos=128)
    toks = synth.tokens_np(S, "toks", S, shape.vocab - 1)[None]
    toks[:, S // 2 + 1:] = shape.mask_id
    lm_pos = np.unique(np.array([0, S // 3, S // 2, S - 1], dtype=np.int32))
    out = model.forward(torch.from_numpy(toks).to(DEV), torch.from_numpy(lm_pos).to(DEV), scale=2.0)
    torch.cuda.synchronize()
    ref = softmax_stats(om.forward_logits(toks, w_np, shape, lm_pos, scale=2.0, mirror=True).reshape(-1, shape.vocab),
                        16)
    print(compare_stats(out.numpy(), ref, 2e-2, max_exceptions=2, id_ranks=4, label=f"bf16 d {d} hd {hd} x {S}"))
    model.close()


# QKV of 64-wide heads in the tiles that the widths above do not reach: 256 x 192
# parts, and 256 x 256 with V^T staged (sequences of whole 64-row tiles) and not
@pytest.mark.parametrize("B_,S", [(1, 130), (6, 427), (41, 64)])
def test_qkv_of_64_wide_heads(P, B_, S):
    shape = ModelShape(n_layers=1, d_model=1536, n_heads=24, head_dim=64, d_ffn=256, vocab=600)
    w_np = synth.model_weights_np(shape, seed=8, dtype="bf16")
    model = P.Model(shape, {k: torch.from_numpy(v).to(DEV).bfloat16() for k, v in w_np.items()}, dtype="bf16",
                    max_pos=512)
    toks = synth.tokens_np(10, "toks", B_ * S, shape.vocab - 1).reshape(B_, S)
    toks[:, S // 2:] = shape.mask_id
    lm_pos = np.unique(np.array([0, S // 3, S // 2, S - 1], dtype=np.int32))
    out = model.forward(torch.from_numpy(toks).to(DEV), torch.from_numpy(lm_pos).to(DEV), scale=2.0)
    torch.cuda.synchronize()
    got, n = out.numpy(), len(lm_pos)
    for b in {0, B_ - 1}:
        ref = softmax_stats(om.forward_logits(toks[b:b + 1], w_np, shape, lm_pos, scale=2.0, mirror=True).reshape(
            -1, shape.vocab), 16)
        print(compare_stats({k: v[b * n:(b + 1) * n] for k, v in got.items()}, ref, 2e-2, max_exceptions=2,
                            id_ranks=4, label=f"bf16 hd 64 {B_} x {S} seq {b}"))
    model.close()


# packed attention: 64 heads x 512 rows is the first size whose 128-query
# workgroups fill the CUs, 64 x 384 takes 32-query ones; blocks smaller than a
# workgroup's queries, and shared rows that end inside one
@pytest.mark.parametrize("S,b0,B,n", [(256, 32, 64, 4), (128, 0, 64, 4), (112, 48, 16, 15)])
def test_packed_attention_layouts(P, S, b0, B, n):
    shape = ModelShape(n_layers=1, d_model=4096, n_heads=64, head_dim=64, d_ffn=128, vocab=500)
    w_np = synth.model_weights_np(shape, seed=5, dtype="f32")
    model = P.Model(shape, {k: torch.from_numpy(v).to(DEV) for k, v in w_np.items()}, dtype="f32", max_pos=256)
    shared = synth.tokens_np(S, "shared", S, shape.vocab - 1)
    shared[b0 + 3:b0 + B] = shape.mask_id
    blocks = np.tile(shared[b0:b0 + B], (n, 1))
    blocks[np.arange(n), 3 + np.arange(n) % (B - 3)] = np.arange(n) + 7
    packed = np.concatenate([shared, blocks.reshape(-1)])
    lm_pos = np.array([b0, b0 + B // 2, b0 + B - 1], dtype=np.int32)
    out = model.forward_packed(torch.from_numpy(packed).to(DEV), S, b0, B, n, torch.from_numpy(lm_pos).to(DEV))
    torch.cuda.synchronize()
    logits = om.packed_logits(packed, w_np, shape, S, b0, B, n, lm_pos)
    print(compare_stats(out.numpy(), softmax_stats(logits.reshape(-1, shape.vocab), 16), 1e-4,
                        label=f"packed S{S} b0{b0} B{B} n{n}"))
    model.close()


# prefix cache writes: a cache off a 16-byte boundary, an offset into it, and
# a length that fills no whole chunk of positions; the rest stays untouched
@pytest.mark.parametrize("S,off,shift", [(37, 0, 0), (300, 5, 0), (64, 3, 1)])
def test_kv_out_alignment(P, S, off, shift):
    from paper_2608_11742_amd._abi import KvCache
    shape = ModelShape(n_layers=2, d_model=256, n_heads=4, head_dim=64, d_ffn=128, vocab=300)
    w_np = synth.model_weights_np(shape, seed=6, dtype="f32")
    model = P.Model(shape, {k: torch.from_numpy(v).to(DEV) for k, v in w_np.items()}, dtype="f32", max_pos=512)
    cap = (off + S + 15) // 8 * 8
    n = shape.n_layers * shape.n_heads * cap * shape.head_dim
    kb, vb = (torch.full((n + 8,), 9.0, device=DEV) for _ in range(2))
    kv = KvCache(kb[shift:].data_ptr(), vb[shift:].data_ptr(), 0, cap)
    toks = synth.tokens_np(9, "t", S, shape.vocab - 1)
    model.forward(torch.from_numpy(toks).to(DEV)[None], torch.zeros(1, dtype=torch.int32, device=DEV), pos_offset=off,
                  kv_out=kv)
    torch.cuda.synchronize()
    got_k = kb[shift:shift + n].cpu().numpy().reshape(2, 4, cap, 64)
    got_v = vb[shift:shift + n].cpu().numpy().reshape(2, 4, 64, cap)
    collect = []
    om.hidden(toks, w_np, shape, pos_offset=off, collect=collect)
    for l, (k, v) in enumerate(collect):
        assert np.allclose(got_k[l, :, off:off + S], k, atol=1e-4)
        assert np.allclose(got_v[l, :, :, off:off + S].transpose(0, 2, 1), v, atol=1e-4)
    rest = np.setdiff1d(np.arange(cap), np.arange(off, off + S))
    assert (got_k[:, :, rest] == 9.0).all() and (got_v[..., rest] == 9.0).all()
    model.close()


# fp32 rounding of the projections, far below the tolerance of a whole forward:
# the kernels and the inputs are fixed, so each figure is too, and each bound
# lies half way between the two it tells apart
def test_f32_swiglu_rounding(P):
    """Gate values reach the output through nothing but the SwiGLU, one
    rounding of the final norm and a factor common to the row: a token's
    embedding is 16 in one place of 256 (its norm exact), attention is switched
    off, the gates of a row are 16 weights of its place, every up is 1 and the
    LM head reads the 16 sums as they are.  The error is 0.765 of 2^-24 (root
    mean square) with a correctly rounded division behind the hardware's
    exponential, 0.839 with the hardware's reciprocal."""
    d, F, V, n = 256, 128, 300, 16
    shape = ModelShape(n_layers=1, d_model=d, n_heads=4, head_dim=64, d_ffn=F, vocab=V, rms_eps=1e-30)
    rng = np.random.default_rng(1)
    w = {"emb": np.zeros((V, d)), "lm_head": np.zeros((V, d)), "layers.0.wqkv": np.zeros((3 * d, d)),
         "layers.0.wo": np.zeros((d, d)), "layers.0.wgu": np.zeros((2 * F, d)), "layers.0.wdown": np.zeros((d, F))}
    rows = np.arange(n, d)                                  # token t: 16 in place t
    w["emb"][rows, rows] = 16.0
    gate = rng.uniform(0.05, 4.0, (n, d)).astype(np.float32)   # 16 x weight: exact
    w["layers.0.wgu"][:n] = gate / 16
    w["layers.0.wgu"][F:F + n] = 1.0 / 16
    w["layers.0.wdown"][np.arange(n), np.arange(n)] = 1.0
    w["lm_head"][np.arange(n), np.arange(n)] = 1.0
    model = P.Model(shape, {k: torch.from_numpy(v.astype(np.float32)).to(DEV) for k, v in w.items()}, dtype="f32",
                    max_pos=256)
    out = model.forward(torch.from_numpy(rows.astype(np.int32)).to(DEV)[None],
                        torch.arange(len(rows), dtype=torch.int32, device=DEV))
    got = out.numpy()["topk_logit"].astype(np.float64)
    g = gate[:, rows].T.astype(np.float64)
    ratio = got / np.sort(g / (1.0 + np.exp(-g)), 1)[:, ::-1]
    err = ratio / ratio.mean(1, keepdims=True) - 1.0        # without the row's own factor
    rms = np.sqrt((err ** 2).mean()) * 2.0 ** 24
    print(f"SwiGLU rounding {rms:.3f}")
    assert rms < 0.80
    model.close()


@pytest.mark.parametrize("B_,S", [(8, 64), (3, 201), (4, 512)])
def test_f32_error_against_64_bits(P, B_, S):
    """Sums over K are folded every 128 values, as K parts of four stages are,
    so that one pass rounds no more than parts do: 2.74e-7, 2.86e-7 and 2.87e-7
    here (2.74e-7, 2.87e-7 and 2.85e-7 in parts), where folds every 256 give
    3.00e-7, 2.95e-7 and 3.19e-7."""
    shape = synth.TINY
    errs = []
    for seed in range(6):
        w_np = synth.model_weights_np(shape, seed=20 + seed, dtype="f32")
        model = P.Model(shape, {k: torch.from_numpy(v).to(DEV) for k, v in w_np.items()}, dtype="f32", max_pos=512)
        toks = synth.tokens_np(21 + seed, "toks", B_ * S, shape.vocab - 1).reshape(B_, S)
        toks[:, S // 2:] = shape.mask_id
        lm_pos = np.arange(S // 2, S, 3, dtype=np.int32)
        out = model.forward(torch.from_numpy(toks).to(DEV), torch.from_numpy(lm_pos).to(DEV))
        got = out.numpy()["topk_logit"][:len(lm_pos)]
        ref = softmax_stats(om.forward_logits(toks[:1], w_np, shape, lm_pos).reshape(-1, shape.vocab), 16).topk_logit
        errs.append(np.linalg.norm(got - ref) / np.linalg.norm(ref))
        model.close()
    print(f"f32 error {B_} x {S}: {np.mean(errs):.3e}", errs)
    assert np.mean(errs) < 2.9e-7


# one workspace, sized for the longest forward of a decode, serves the shorter
# ones: few rows take more K parts and smaller LM head tiles than many
def test_workspace_serves_every_smaller_forward(P):
    shape = ModelShape(n_layers=1, d_model=2048, n_heads=32, head_dim=64, d_ffn=5632, vocab=4000)
    gen = torch.Generator(device=DEV).manual_seed(1)
    dims = {"emb": (4000, 2048), "lm_head": (4000, 2048), "layers.0.wqkv": (6144, 2048), "layers.0.wo": (2048, 2048),
            "layers.0.wgu": (11264, 2048), "layers.0.wdown": (2048, 5632)}
    w = {k: torch.empty(s, dtype=torch.bfloat16, device=DEV).normal_(0, 0.02, generator=gen) for k, s in dims.items()}
    model = P.Model(shape, w, dtype="bf16", max_pos=1024)
    need = lambda b, s, n: P.dllm_workspace_bytes(model.handle, b, s, n)
    for b, n in [(1, 300), (1, 1), (3, 64)]:
        sizes = [need(b, s, min(n, s)) for s in range(1, 1025)]
        assert sizes == sorted(sizes)
    packed = [P.dllm_workspace_bytes_packed(model.handle, 256, 32, n, 32) for n in range(16)]
    assert packed == sorted(packed)
    assert need(1 << 20, 1 << 20, 1 << 20) > 0      # past every limit: an answer all the same
    ws = torch.empty(need(1, 1024, 300), dtype=torch.uint8, device=DEV)
    for s in (17, 33, 129, 257, 300, 321, 513, 769, 1023):
        n = min(s, 300)
        toks = torch.from_numpy(synth.tokens_np(s, "t", s, 3999)).to(DEV)[None]
        lm = torch.arange(n, dtype=torch.int32, device=DEV)
        out, own = P.Stats(n, 16, device=DEV), P.Stats(n, 16, device=DEV)
        P.dllm_forward(model.handle, toks, lm, out, ws)
        P.dllm_forward(model.handle, toks, lm, own, torch.empty(need(1, s, n), dtype=torch.uint8, device=DEV))
        for k, v in out.numpy().items():
            assert np.array_equal(v, own.numpy()[k]), (s, k)
    model.close()
