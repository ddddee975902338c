"""Attention with 32 query rows per wave: which calls take it (a table of many tokens and more than 80 rows per KV head) and,
at the edges of its blocks, ring, row chunks and page lookups, its results against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from helpers import rel_err, to_np_f32
from paper_2402_11131_amd import api, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = {
    # B, H, Hkv, page, T, gamma, tokens of the table, lens, forced split length
    "cut_five_chunks": (2, 8, 2, 64, 32, 4, 61440, [1500, 400], 0),           # 640 rows = 5 x 128, cut on the device
    "cut_empty": (3, 4, 1, 16, 24, 4, 150016, [0, 31, 33], 0),                # 480 rows = 5 x 96
    "cut_many_new_rows": (2, 4, 1, 32, 64, 8, 36864, [700, 64], 0),           # 2304 rows, 18 blocks of new rows
    "forced_splits": (2, 8, 2, 16, 24, 4, 61440, [2100, 129], 96),            # 480 rows, three blocks per split, merge kernel
    "forced_ring": (5, 4, 1, 32, 32, 4, 61440, [1, 32, 96, 127, 128], 61440), # 640 rows, unsplit: fewer blocks than the ring
    "unsplit": (8, 64, 32, 64, 32, 2, 2432, [2176, 2432, 2047, 31, 0, 97, 1000, 64], 0),   # 192 rows = 2 x 96, 68 and 76 blocks
    "one_chunk": (4, 8, 8, 16, 24, 3, 38400, [300, 2100, 95, 0], 0),          # 96 rows, streamed
    "one_chunk_unsplit": (16, 32, 32, 32, 12, 6, 2400, [2400] + [97 * i for i in range(15)], 0),   # 84 rows of 96
}


def _inputs(name):
    B, H, Hkv, page, T, gamma, cap, lens, split = CASES[name]
    cfg = synth.scaled(synth.CONFIGS["c2"], B=B, H=H, Hkv=Hkv, D=128, page=page, T=T, gamma=gamma, branching=(8, 8, 4),
                       max_depth=3, L_min=max(lens), L_max=max(lens))
    inp = synth.make_msa_inputs(cfg, 5)
    inp["seq_lens"] = torch.tensor(lens, dtype=torch.int32)
    table = torch.zeros(B, cap // page, dtype=torch.int32)
    table[:, :inp["block_table"].shape[1]] = inp["block_table"]
    inp["block_table"] = table
    return cfg, inp


def _rows_per_wave(cfg, cap, workspace_bytes=None):
    return api.ss_msa_plan_launch(cfg.B, cfg.T, cfg.gamma, cfg.H, cfg.Hkv, cfg.D, cap, workspace_bytes)["rows_per_wave"]


def _run(inp, cfg, split=0, rows_per_wave=32, **kw):
    """The call, which has to take the kernel with that many query rows per wave."""
    d = {k: (v.to(DEV) if isinstance(v, torch.Tensor) else v) for k, v in inp.items()}
    ws = kw.get("workspace")
    prev = api.ss_msa_set_split_keys(split)
    try:
        assert _rows_per_wave(cfg, d["block_table"].shape[1] * cfg.page, None if ws is None else ws.numel()) == rows_per_wave
        got = api.ss_msa_attention(d["q"], d["k_new"], d["v_new"], d["k_cache"], d["v_cache"], d["block_table"], d["seq_lens"],
                                   d["parent"], cfg.gamma, d["scale"], out=torch.full_like(d["q"], 3.0), **kw)
    finally:
        api.ss_msa_set_split_keys(prev)
    torch.cuda.synchronize()
    return got


def _check(got, inp, cfg, flags=0, nodes=None):
    a = [to_np_f32(inp[k]) for k in ("q", "k_new", "v_new", "k_cache", "v_cache")]
    a += [inp["block_table"].numpy(), inp["seq_lens"].numpy(), inp["parent"].numpy(), cfg.gamma, inp["scale"]]
    want = oracle.msa_attention(*a, flags=flags) if nodes is None else oracle.msa_attention_pruned(*a, nodes.numpy())
    keep = np.ones(cfg.B * cfg.R, bool)
    if nodes is not None:
        keep[:] = False
        keep[oracle.live_rows(nodes.numpy(), cfg.T, cfg.gamma)] = True
        assert bool((got.view(cfg.B * cfg.R, -1)[torch.from_numpy(~keep).to(DEV)] == 3.0).all())
    keep = keep.reshape(cfg.B, cfg.R)
    # 2e-2 is the bf16 path's tolerance; rows of few keys average nothing out: bf16 probabilities and the rounding of the
    # result, 2^-9 each in numerator, denominator and result, of the largest value (a twentieth more for the second order)
    few = 1.05 * 3 * 2.0 ** -9 * float(inp["v_new"].float().abs().max())
    for b in range(cfg.B):
        g, w = to_np_f32(got[b])[keep[b]], want[b][keep[b]]
        assert np.isfinite(g).all()
        assert rel_err(g, w) <= 2e-2 or (int(inp["seq_lens"][b]) < 64 and np.abs(g - w).max() <= few), (b, rel_err(g, w))


@pytest.mark.parametrize("pruned", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_against_the_oracle(name, pruned):
    cfg, inp = _inputs(name)
    nodes = None
    if pruned:
        nodes = torch.tensor([1 + (i * 7 + 3) % cfg.T for i in range(cfg.B)], dtype=torch.int32)
        for b in range(cfg.B):
            inp["parent"][b, int(nodes[b]):] = 0
    split = CASES[name][8]
    got = _run(inp, cfg, split, **({} if nodes is None else dict(n_nodes=nodes.to(DEV))))
    _check(got, inp, cfg, nodes=nodes)


@pytest.mark.parametrize("name", ["cut_five_chunks", "unsplit", "one_chunk"])
def test_streams_that_do_not_see_themselves(name):
    cfg, inp = _inputs(name)
    _check(_run(inp, cfg, flags=api.SS_STREAM_EXCLUDE_SELF), inp, cfg, flags=api.SS_STREAM_EXCLUDE_SELF)


@pytest.mark.parametrize("name", ["forced_ring", "unsplit"])
def test_running_maximum_that_keeps_moving(name):
    # every block's scores outgrow the ones before by more than 2^16, then fall: the sums are brought down many times
    cfg, inp = _inputs(name)
    for b, n in enumerate(CASES[name][7]):
        for t in range(n):
            page, slot = int(inp["block_table"][b, t // cfg.page]), t % cfg.page
            inp["k_cache"][page, :, slot] *= 1.0 + (t // 32 if t < 1024 else 0)
    inp["q"] *= 8
    _check(_run(inp, cfg, CASES[name][8]), inp, cfg)


def test_memory_past_the_end_may_hold_nan():
    cfg, inp = _inputs("unsplit")
    base = _run(inp, cfg)
    used = torch.zeros(inp["k_cache"].shape[0], cfg.page, dtype=torch.bool)
    for b, n in enumerate(CASES["unsplit"][7]):
        for t in range(n):
            used[int(inp["block_table"][b, t // cfg.page]), t % cfg.page] = True
    page, slot = (~used).nonzero(as_tuple=True)
    inp["k_cache"][page, :, slot] = float("nan")
    inp["v_cache"][page, :, :, slot] = float("nan")
    assert torch.equal(_run(inp, cfg), base)


@pytest.mark.parametrize("name", ["cut_five_chunks", "one_chunk"])
def test_a_workspace_for_the_other_kernel_is_taken_as_before(name):
    # the call falls back to 16 rows per wave where only that kernel's splits fit; both round bf16 probabilities and outputs
    cfg, inp = _inputs(name)
    full = api.ss_msa_workspace_bytes(cfg.B, cfg.T, cfg.gamma, cfg.H, cfg.Hkv, cfg.D, CASES[name][6], api.SS_BF16)
    want = _run(inp, cfg)
    zeros = lambda n: torch.zeros(n, dtype=torch.uint8, device=DEV)
    assert torch.equal(_run(inp, cfg, workspace=zeros(full)), want)
    got = _run(inp, cfg, workspace=zeros(full - 1), rows_per_wave=16)
    assert not torch.equal(got, want)
    assert (got.float() - want.float()).norm() <= 2.0 ** -7 * want.float().norm()
    _check(got, inp, cfg)
    few = full - 1                      # the least that the other kernel's splits fit, and a byte less
    lo = 0
    while few - lo > 1:
        mid = (few + lo) // 2
        try:
            _rows_per_wave(cfg, CASES[name][6], mid)
            few = mid
        except api.SSError:
            lo = mid
    assert torch.equal(_run(inp, cfg, workspace=zeros(few), rows_per_wave=16), got)
    with pytest.raises(api.SSError) as e:
        api.ss_msa_plan_launch(cfg.B, cfg.T, cfg.gamma, cfg.H, cfg.Hkv, cfg.D, CASES[name][6], few - 1)
    assert e.value.code == 4


def test_which_calls_take_it():
    # two workgroups per compute unit make more splits of a batch that does not fill them
    rows = lambda B, T, g, Hkv, D, cap: api.ss_msa_plan_launch(B, T, 4, Hkv * g, Hkv, D, cap)["rows_per_wave"]
    assert rows(4, 32, 4, 8, 128, 8192) == 32 and rows(4, 32, 4, 8, 128, 4096) == 16
    assert rows(4, 32, 4, 8, 64, 8192) == 16 and rows(4, 16, 4, 8, 128, 16384) == 16
    plan = lambda B, T, g, Hkv, D, cap: api.ss_msa_plan(B, T, 4, Hkv * g, Hkv, D, cap, api.SS_BF16)
    assert plan(4, 32, 4, 8, 128, 8192) == (3, 2)      # 640 rows, 80 blocks per workgroup in flight
    assert plan(4, 32, 4, 8, 128, 4096) == (2, 1)      # 40: 16 rows per wave, two splits merged in the kernel
    assert plan(4, 32, 4, 8, 64, 8192) == (2, 1)       # heads of 64
    assert plan(4, 16, 4, 8, 128, 16384) == (2, 1)     # 320 rows pad to 384


def test_the_call_without_a_workspace_has_the_same_plan():
    # four splits of 9600 tokens: 32.25 MiB of partial results, and 16.1 MiB with 16 rows per wave
    B, T, gamma, H, Hkv, cap = 4, 32, 3, 32, 8, 9600
    p = api.ss_msa_plan_launch(B, T, gamma, H, Hkv, 128, cap)
    need = api.ss_msa_workspace_bytes(B, T, gamma, H, Hkv, 128, cap, api.SS_BF16)
    limit = api.ss_msa_static_scratch_bytes()
    assert (p["rows_per_wave"], p["n_splits"]) == (32, 4) and need > limit + 262144
    less = api.ss_msa_plan_launch(B, T, gamma, H, Hkv, 128, cap, limit)
    assert (less["rows_per_wave"], less["n_splits"]) == (16, 2)
    cfg = synth.scaled(synth.CONFIGS["c2"], B=B, H=H, Hkv=Hkv, D=128, page=64, T=T, gamma=gamma, branching=(8, 8, 4), max_depth=3,
                       L_min=300, L_max=700)
    inp = synth.make_msa_inputs(cfg, 5)
    table = torch.zeros(B, cap // 64, dtype=torch.int32)
    table[:, :inp["block_table"].shape[1]] = inp["block_table"]
    inp["block_table"] = table
    want = _run(inp, cfg)
    d = {k: (v.to(DEV) if isinstance(v, torch.Tensor) else v) for k, v in inp.items()}
    got = api.ss_msa_attention_static(d["q"], d["k_new"], d["v_new"], d["k_cache"], d["v_cache"], d["block_table"], d["seq_lens"],
                                      d["parent"], gamma, d["scale"], out=torch.full_like(d["q"], 3.0))
    assert torch.equal(got, want)
    _check(got, inp, cfg)
