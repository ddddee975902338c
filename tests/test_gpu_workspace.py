"""One workspace, zeroed once, serves calls of any shape it is large enough for: shapes whose splits are merged inside
the attention kernel (arrival counters in the workspace) alternate with each other and with shapes that leave partial
rows and a table of cuts there."""
import pytest
import torch

from paper_2402_11131_amd import api, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = {
    # dtype, B, H, Hkv, D, page, T, gamma, cached tokens, block-table columns over the needed ones
    "two_splits_large": ("bf16", 4, 32, 32, 64, 16, 16, 4, 1024, 1),
    "two_splits_small": ("bf16", 4, 32, 32, 64, 16, 8, 4, 1024, 1),
    "two_splits_batch_5": ("bf16", 5, 32, 32, 64, 16, 8, 2, 700, 1),
    "merge_kernel": ("bf16", 1, 32, 32, 64, 16, 16, 4, 2048, 1),
    "cut_on_the_device": ("bf16", 3, 8, 2, 64, 64, 24, 3, 700, 32),
    "fp32": ("f32", 1, 4, 4, 64, 16, 8, 3, 1024, 1),
}


def _args(name):
    dt, B, H, Hkv, D, page, T, gamma, L, wide = SHAPES[name]
    cfg = synth.scaled(synth.CONFIGS["c2"], B=B, H=H, Hkv=Hkv, D=D, page=page, T=T, gamma=gamma, branching=(8, 8), max_depth=2,
                       L_min=L, L_max=L, dtype=dt)
    d = {k: (v.to(DEV) if isinstance(v, torch.Tensor) else v) for k, v in synth.make_msa_inputs(cfg, 3).items()}
    table = torch.zeros(B, d["block_table"].shape[1] * wide, dtype=torch.int32, device=DEV)
    table[:, :d["block_table"].shape[1]] = d["block_table"]
    code = api.SS_F32 if dt == "f32" else api.SS_BF16
    shape = (B, T, gamma, H, Hkv, D, table.shape[1] * page, code)
    return shape, (d["q"], d["k_new"], d["v_new"], d["k_cache"], d["v_cache"], table, d["seq_lens"], d["parent"], gamma, d["scale"])


def test_shapes_alternate_in_one_workspace():
    calls = {n: _args(n) for n in SHAPES}
    assert [api.ss_msa_plan(*calls[n][0]) for n in SHAPES][:3] == [(2, 1)] * 3          # merged in the attention kernel
    shape, args = calls["cut_on_the_device"]
    assert api.ss_msa_plan_splits(*shape, args[6].tolist())[0] == 2
    need = max(api.ss_msa_workspace_bytes(*shape) for shape, _ in calls.values())
    ws = api.ss_msa_workspace_init(torch.empty(need, dtype=torch.uint8, device=DEV))
    want = {n: api.ss_msa_attention(*args) for n, (_, args) in calls.items()}           # a fresh workspace each
    order = ["two_splits_large", "two_splits_small", "two_splits_large", "merge_kernel", "two_splits_small", "two_splits_batch_5",
             "cut_on_the_device", "two_splits_small", "fp32", "two_splits_batch_5", "two_splits_large", "cut_on_the_device"]
    for n in order:
        args = calls[n][1]
        got = api.ss_msa_attention(*args, out=torch.full_like(args[0], 3.0), workspace=ws)
        assert torch.equal(got, want[n]), n
