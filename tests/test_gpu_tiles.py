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
