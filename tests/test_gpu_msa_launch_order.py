"""Launches of ten and twelve waves (heads of 64) and more workgroups than compute units, whose workgroups come in order of the splits: batches of
full, partly filled and empty tables against the oracle, with groups that are no multiple of eight, and bit for bit what the
attention and the merge kernel give as two calls."""
import numpy as np
import pytest
import torch

import oracle
from helpers import rel_err, to_np_f32
from paper_2402_11131_amd import api, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = {
    # B, H, Hkv, T, gamma, page, tokens of the table, lens -> waves, splits, workgroups
    "three_chunks": (3, 15, 5, 12, 4, 16, 1536, [1536, 700, 33], 12, 6, 288),
    "two_splits": (3, 27, 27, 32, 5, 64, 768, [768, 0, 385], 12, 2, 504),
    "one_split": (10, 18, 9, 16, 5, 32, 480, [480, 479, 1, 0, 31, 32, 33, 300, 64, 17], 12, 1, 288),
    "one_chunk": (3, 30, 30, 12, 5, 16, 1024, [1024, 340, 0], 10, 3, 272),
}


@pytest.mark.parametrize("name", list(CASES))
def test_order_of_the_splits(name):
    B, H, Hkv, T, gamma, page, cap, lens, waves, splits, wgs = CASES[name]
    p = api.ss_msa_plan_launch(B, T, gamma, H, Hkv, 64, cap)
    assert (p["waves"], p["n_splits"], p["workgroups"]) == (waves, splits, wgs)
    cfg = synth.scaled(synth.CONFIGS["c2"], B=B, H=H, Hkv=Hkv, D=64, page=page, T=T, gamma=gamma, branching=(4, 4, 4), max_depth=3,
                       L_min=cap, L_max=cap)
    inp = synth.make_msa_inputs(cfg, 7)
    d = {k: (v.to(DEV) if isinstance(v, torch.Tensor) else v) for k, v in inp.items()}
    ws = api.ss_msa_workspace(B, T, gamma, H, Hkv, 64, cap, api.SS_BF16, DEV)

    def call(lens, **kw):
        return api.ss_msa_attention(d["q"], d["k_new"], d["v_new"], d["k_cache"], d["v_cache"], d["block_table"],
                                    torch.tensor(lens, dtype=torch.int32, device=DEV), d["parent"], gamma, d["scale"],
                                    workspace=ws, **kw)
    a = [to_np_f32(inp[k]) for k in ("q", "k_new", "v_new", "k_cache", "v_cache")]
    few = 1.05 * 3 * 2.0 ** -9 * float(d["v_new"].float().abs().max())   # rows of few keys average nothing out (see test_gpu_msa_uneven)
    for n in (lens, [cap] * B, lens[::-1]):
        got = call(n)
        if splits > 1:
            two = torch.zeros_like(got)
            call(n, out=two, flags=api.SS_MSA_PARTIALS_ONLY)
            call(n, out=two, flags=api.SS_MSA_MERGE_ONLY)
            assert torch.equal(got, two), n
        want = oracle.msa_attention(*a, inp["block_table"].numpy(), np.array(n, np.int32), inp["parent"].numpy(), gamma, inp["scale"])
        for b in range(B):
            g, w = to_np_f32(got[b]), want[b]
            assert rel_err(g, w) <= 2e-2 or (n[b] < 64 and np.abs(g - w).max() <= few), (n, b)
