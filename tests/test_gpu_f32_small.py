"""fp32 kernels at the edges of their tiles: workgroups of 4 rows (up to 256 of 8 would be made) and of 8 with a ragged last
one, key tiles of 64 that end before, at and after the prefix, an empty prefix; the LM head's selection among equal,
infinite and NaN logits in tiles narrower than K.  Against the oracle, with the tolerance of test_gpu_msa.py."""
import numpy as np
import pytest
import torch

import oracle
from helpers import rel_err, to_np_f32
from paper_2402_11131_amd import api, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = {
    # B, H, Hkv, D, T, gamma, lens
    "one_row": (1, 2, 1, 64, 1, 0, [1]),
    "five_rows": (3, 4, 2, 64, 1, 4, [0, 63, 64]),
    "tiles": (4, 4, 4, 64, 11, 2, [65, 127, 128, 193]),
    "at_256": (8, 8, 8, 64, 8, 3, [100, 60, 0, 130, 7, 64, 1, 129]),
    "past_256": (8, 8, 8, 64, 11, 2, [100, 60, 0, 130, 7, 64, 1, 129]),
    "wide_heads": (2, 4, 2, 128, 7, 2, [0, 130]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_attention(name):
    B, H, Hkv, D, T, gamma, lens = CASES[name]
    cap = max(lens)
    cfg = synth.scaled(synth.CONFIGS["c1"], B=B, H=H, Hkv=Hkv, D=D, page=16, T=T, gamma=gamma, branching=(4, 4), max_depth=2, L_min=cap, L_max=cap)
    inp = synth.make_msa_inputs(cfg, 6)
    assert inp["q"].dtype == torch.float32
    d = {k: (v.to(DEV) if isinstance(v, torch.Tensor) else v) for k, v in inp.items()}
    got = api.ss_msa_attention(d["q"], d["k_new"], d["v_new"], d["k_cache"], d["v_cache"], d["block_table"],
                               torch.tensor(lens, dtype=torch.int32, device=DEV), d["parent"], gamma, d["scale"])
    want = oracle.msa_attention(*[to_np_f32(inp[k]) for k in ("q", "k_new", "v_new", "k_cache", "v_cache")],
                                inp["block_table"].numpy(), np.array(lens, np.int32), inp["parent"].numpy(), gamma, inp["scale"])
    for b in range(B):
        assert rel_err(to_np_f32(got[b]), want[b]) <= 1e-5, b


@pytest.mark.parametrize("N", [1, 5, 9])
def test_selection(N):
    V, d, K = 66, 8, 4   # the second tile of 64 ids holds two
    h = torch.zeros(N, d)
    h[:, 0] = 1.0
    W = torch.zeros(V, d)
    W[:, 0] = torch.arange(V) // 7 * 0.5 - 1.0      # runs of equal logits
    W[3, 0], W[9, 0] = float("inf"), float("-inf")
    idx, val = api.ss_lm_head_argmax_topk(h.cuda(), W.cuda(), K)
    logits = W[:, 0]
    want = sorted(range(V), key=lambda i: (-float(logits[i]), i))[:K]
    assert idx.cpu().tolist() == [want] * N and val.cpu().tolist() == [[float(logits[i]) for i in want]] * N
    W[64:, 0] = float("nan")                         # never selected
    W[3, 0] = 2.0
    idx, _ = api.ss_lm_head_argmax_topk(h.cuda(), W.cuda(), K)
    ok = [i for i in range(64)]
    assert idx.cpu().tolist() == [sorted(ok, key=lambda i: (-float(W[i, 0]), i))[:K]] * N
