"""The fp32 kernels on both sides of their choice of rows per workgroup, with remainders of every tile."""
import numpy as np
import pytest
import torch

import oracle
from helpers import rel_err, to_np_f32
from paper_2402_11131_amd import api, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# Heads of 64: 511 workgroups of 32 rows (chunks, splits and heads) are cut into smaller ones, 512 and more are not
@pytest.mark.parametrize("B,H,R,L,keys,wgs", [(7, 73, 32, 70, 0, 511), (8, 64, 32, 70, 0, 512), (4, 16, 32, 448, 64, 448), (4, 16, 32, 512, 64, 512),
                                             (4, 16, 33, 193, 64, 512), (3, 9, 33, 500, 64, 432)])
def test_attention_at_the_choice_of_rows(B, H, R, L, keys, wgs):
    before = api.ss_msa_set_split_keys(keys)
    try:
        n, _ = api.ss_msa_plan(B, R, 0, H, H, 64, -(-L // 16) * 16, api.SS_F32)
        assert B * H * -(-R // 32) * n == wgs
        test_attention(B, H, H, 64, R, 0, L)
    finally:
        api.ss_msa_set_split_keys(before)


@pytest.mark.parametrize("B,H,Hkv,D,T,gamma,L", [(4, 16, 4, 64, 8, 3, 70), (5, 13, 13, 64, 8, 3, 70), (2, 4, 2, 128, 11, 2, 1),
                                                 (9, 4, 4, 128, 17, 1, 129), (1, 2, 1, 128, 1, 0, 0), (3, 4, 4, 64, 5, 1, 700)])
def test_attention(B, H, Hkv, D, T, gamma, L):
    cfg = synth.scaled(synth.CONFIGS["c1"], B=B, H=H, Hkv=Hkv, D=D, T=T, gamma=gamma, branching=(8, 8), max_depth=2, L_min=L, L_max=L)
    inp = synth.make_msa_inputs(cfg, 3)
    d = {k: (v.to(DEV) if isinstance(v, torch.Tensor) else v) for k, v in inp.items()}
    got = api.ss_msa_attention(d["q"], d["k_new"], d["v_new"], d["k_cache"], d["v_cache"], d["block_table"], d["seq_lens"],
                               d["parent"], gamma, d["scale"])
    want = oracle.msa_attention(*[to_np_f32(inp[k]) for k in ("q", "k_new", "v_new", "k_cache", "v_cache")],
                                inp["block_table"].numpy(), inp["seq_lens"].numpy(), inp["parent"].numpy(), gamma, inp["scale"])
    assert rel_err(to_np_f32(got), want) <= 1e-5     # the fp32 path's tolerance


# Features and ids with remainders
@pytest.mark.parametrize("N,d,V", [(1, 1, 1), (7, 63, 65), (33, 65, 64 * 127 + 1), (32, 64, 64 * 255), (32, 64, 64 * 255 + 1), (70, 130, 6000)])
def test_projection(N, d, V):
    rng = synth.rng_for(N + d + V)
    x, W = rng.standard_normal((N, d), np.float32), rng.standard_normal((V, d), np.float32)
    got = api.ss_linear_rows(torch.from_numpy(x).to(DEV), torch.from_numpy(W).to(DEV), torch.empty(N, V, device=DEV)).cpu().numpy()
    want = x.astype(np.float64) @ W.astype(np.float64).T
    bound = (d + 1) * 2.0 ** -24 * (np.abs(x).astype(np.float64) @ np.abs(W).astype(np.float64).T)   # d rounded steps
    assert (np.abs(got - want) <= bound).all()


# 3200 workgroups of eight rows and one more; of listed rows the launch is shaped for plan_rows, whatever their number
@pytest.mark.parametrize("N,V,plan,live", [(64, 64 * 400, 64, 64), (64, 64 * 400 + 1, 64, 64), (8, 64 * 3201, 8, 8), (70, 6400, 8, 70), (70, 6400, 70, 9),
                                           (300, 64 * 100, 40, 33)])
def test_projection_of_listed_rows(N, V, plan, live):
    d = 67
    rng = synth.rng_for(N + V + plan)
    x, W = rng.standard_normal((N, d), np.float32), rng.standard_normal((V, d), np.float32)
    rows = np.sort(rng.permutation(N)[:live]).astype(np.int32)
    listed = torch.zeros(N, dtype=torch.int32)
    listed[:live] = torch.from_numpy(rows)
    y = torch.full((N, V), 3.0, device=DEV)
    api.ss_linear_rows(torch.from_numpy(x).to(DEV), torch.from_numpy(W).to(DEV), y, plan_rows=plan,
                       live=(listed.to(DEV), torch.tensor([live], dtype=torch.int32, device=DEV)))
    got = y.cpu().numpy()
    want = x[rows].astype(np.float64) @ W.astype(np.float64).T
    bound = (d + 1) * 2.0 ** -24 * (np.abs(x[rows]).astype(np.float64) @ np.abs(W).astype(np.float64).T)   # d rounded steps
    assert (np.abs(got[rows] - want) <= bound).all()
    assert (np.delete(got, rows, axis=0) == 3.0).all()
