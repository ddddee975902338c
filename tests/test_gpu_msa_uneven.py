"""Attention over batches whose lengths do not fill the block table.  Launches with several row chunks (the query heads
of a KV head times the tree's rows beyond 80) and long splits by the host's plan are cut into splits on the device; the
others keep the host's cut.  Both kinds, and that every shape is of the kind it stands for, against the oracle (large
shapes: against the host's cut, forced), full and pruned trees, one call and two."""
import numpy as np
import pytest
import torch

import oracle
from helpers import rel_err, to_np_f32
from paper_2402_11131_amd import api, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = {
    # B, H, Hkv, D, page, T, gamma, lens, columns of the table over the longest sequence's, large
    # the host's cut: one row chunk, or splits below 1024 tokens, or more sequences than a wave has lanes
    "one_short": (1, 4, 1, 128, 16, 5, 1, [300], 6.0, False),
    "empty_and_odd_heads": (3, 6, 3, 64, 32, 8, 3, [1200, 0, 77], 1.0, False),
    "merged_in_kernel": (4, 32, 32, 64, 16, 3, 1, [2000, 700, 31, 1500], 1.5, False),
    "all_lanes": (64, 2, 2, 64, 16, 2, 1, [(i * 37) % 600 for i in range(64)], 1.0, False),
    "more_than_lanes": (65, 2, 2, 64, 16, 2, 1, [(i * 37) % 600 for i in range(65)], 1.0, False),
    "short_chunks_merged_in_kernel": (4, 48, 16, 64, 16, 16, 2, [1100, 513, 0, 700], 1.0, False),
    "short_chunks_all_lanes": (64, 4, 1, 64, 16, 8, 2, [(i * 37) % 600 for i in range(64)], 1.0, False),
    "chunks_more_than_lanes": (65, 4, 1, 64, 16, 8, 2, [(i * 37) % 600 for i in range(65)], 4.0, False),
    "short_chunks_three_kv_heads": (3, 12, 3, 128, 32, 8, 3, [1200, 0, 77], 1.5, False),
    "short_row_chunks": (2, 8, 1, 128, 64, 24, 3, [1500, 400], 2.0, False),
    "new_rows_longer_than_a_short_split": (2, 4, 2, 64, 16, 64, 8, [700, 300], 2.0, False),
    # cut on the device: a table much wider than the lengths gives the host's plan long splits
    "cut_merged_in_kernel": (4, 48, 16, 64, 16, 16, 2, [1100, 513, 0, 700], 3.0, False),     # 3 chunks of 48 rows
    "cut_all_lanes": (64, 4, 1, 64, 16, 8, 2, [2300] + [(i * 37) % 600 for i in range(63)], 1.0, False),  # 2 of 48, merged likewise
    "cut_three_kv_heads": (3, 18, 3, 128, 32, 8, 3, [1200, 0, 77], 25.0, False),             # 3 of 64
    "cut_five_waves": (2, 20, 5, 128, 64, 8, 4, [1500, 400], 20.0, False),                   # 2 of 80
    "cut_eight_waves": (2, 8, 1, 128, 64, 24, 3, [1500, 400], 30.0, False),                  # 6 of 128
    "cut_new_rows_longer_than_a_split": (2, 4, 2, 64, 16, 64, 8, [700, 300], 20.0, False),   # 9 of 128
    "cut_more_splits_than_the_host": (2, 12, 2, 64, 16, 32, 2, [9000, 1], 1.0, False),
    "many_rounds": (8, 32, 8, 128, 64, 32, 4, [2000, 8192, 3000, 5000, 2500, 33, 7000, 4097], 1.0, True),
}
CUT = [n for n in CASES if n.startswith("cut_")] + ["many_rounds"]


def _shape(name):
    B, H, Hkv, D, page, T, gamma, lens, room, _ = CASES[name]
    return B, T, gamma, H, Hkv, D, int((max(lens) + page - 1) // page * room) * page, api.SS_BF16


def _inputs(name, device=None):
    """Configuration and (q, k_new, v_new, k_cache, v_cache, block_table, seq_lens, parent, gamma, scale) on the GPU, and on
    the CPU if the oracle is to have them."""
    B, H, Hkv, D, page, T, gamma, lens, room, large = CASES[name]
    cfg = synth.scaled(synth.CONFIGS["c2"], B=B, H=H, Hkv=Hkv, D=D, page=page, T=T, gamma=gamma, branching=(8, 8),
                       max_depth=2, L_min=max(lens), L_max=max(lens))
    inp = synth.make_msa_inputs(cfg, 5, device=DEV if large else None)
    d = {k: (v.to(DEV) if isinstance(v, torch.Tensor) else v) for k, v in inp.items()}
    d["seq_lens"] = torch.tensor(lens, dtype=torch.int32, device=DEV)
    table = d["block_table"]
    d["block_table"] = torch.zeros(B, _shape(name)[6] // page, dtype=torch.int32, device=DEV)
    d["block_table"][:, :table.shape[1]] = table
    return cfg, inp, d


@pytest.mark.parametrize("pruned", [False, True])
@pytest.mark.parametrize("name", list(CASES))
def test_uneven_batches(name, pruned):
    B, H, Hkv, D, page, T, gamma, lens, room, large = CASES[name]
    cfg, inp, d = _inputs(name)
    nodes = torch.tensor([1 + (i * 5) % T for i in range(B)], dtype=torch.int32) if pruned else None
    parent = d["parent"].clone()
    if pruned:
        for b in range(B):
            parent[b, int(nodes[b]):] = 0
    where, _ = api.ss_msa_plan_splits(*_shape(name), lens, nodes.tolist() if pruned else None)
    assert where == (2 if name in CUT else 0)
    args = (d["q"], d["k_new"], d["v_new"], d["k_cache"], d["v_cache"], d["block_table"], d["seq_lens"], parent, gamma, d["scale"])
    kw = dict(n_nodes=nodes.to(DEV)) if pruned else {}
    got = api.ss_msa_attention(*args, out=torch.full_like(d["q"], 3.0), **kw)
    # the two kernels as two calls give the same bits
    ws = api.ss_msa_workspace(B, T, gamma, H, Hkv, D, d["block_table"].shape[1] * page, api.SS_BF16, DEV)
    two = torch.full_like(d["q"], 3.0)
    merge_kernel = api.ss_msa_plan(B, T, gamma, H, Hkv, D, d["block_table"].shape[1] * page, api.SS_BF16)[0] > 1
    api.ss_msa_attention(*args, out=two, workspace=ws, flags=api.SS_MSA_PARTIALS_ONLY, **kw)
    if merge_kernel:
        api.ss_msa_attention(*args, out=two, workspace=ws, flags=api.SS_MSA_MERGE_ONLY, **kw)
    torch.cuda.synchronize()
    assert torch.equal(got, two)
    if large:
        prev = api.ss_msa_set_split_keys(1024)
        try:
            want = to_np_f32(api.ss_msa_attention(*args, out=torch.full_like(d["q"], 3.0), **kw))
        finally:
            api.ss_msa_set_split_keys(prev)
    else:
        a = [to_np_f32(inp[k]) for k in ("q", "k_new", "v_new", "k_cache", "v_cache")]
        a += [d["block_table"].cpu().numpy(), np.array(lens, np.int32), parent.cpu().numpy(), gamma, inp["scale"]]
        want = oracle.msa_attention_pruned(*a, nodes.numpy()) if pruned else oracle.msa_attention(*a)
    keep = np.ones(B * cfg.R, bool)
    if pruned:
        keep[:] = False
        keep[oracle.live_rows(nodes.numpy(), T, gamma)] = True
        assert bool((got.view(B * cfg.R, -1)[torch.from_numpy(~keep).to(DEV)] == 3.0).all())
    keep = keep.reshape(B, cfg.R)
    # Per sequence, for a short one's values are many times a long one's.  2e-2 is the bf16 path's tolerance; a row of
    # few keys averages nothing out, so for short sequences the bound counts: bf16 probabilities (2^-9 each, in the
    # sum over the values and in the sum they are divided by) and the rounding of the result, 3 * 2^-9 of the largest
    # value; a twentieth more for the second order.
    few = 1.05 * 3 * 2.0 ** -9 * float(d["v_new"].float().abs().max())
    for b in range(B):
        g, w = to_np_f32(got[b])[keep[b]], want[b][keep[b]]
        assert rel_err(g, w) <= 2e-2 or (lens[b] < 64 and np.abs(g - w).max() <= few), (b, rel_err(g, w))


def _args(d, parent=None):
    return (d["q"], d["k_new"], d["v_new"], d["k_cache"], d["v_cache"], d["block_table"], d["seq_lens"], d["parent"])


@pytest.mark.parametrize("name", ["cut_merged_in_kernel", "cut_three_kv_heads"])
def test_streams_that_do_not_see_themselves(name):
    cfg, inp, d = _inputs(name)
    got = api.ss_msa_attention(*_args(d), cfg.gamma, inp["scale"], flags=api.SS_STREAM_EXCLUDE_SELF)
    a = [to_np_f32(inp[k]) for k in ("q", "k_new", "v_new", "k_cache", "v_cache")]
    want = oracle.msa_attention(*a, d["block_table"].cpu().numpy(), d["seq_lens"].cpu().numpy(), d["parent"].cpu().numpy(),
                                cfg.gamma, inp["scale"], flags=api.SS_STREAM_EXCLUDE_SELF)
    long = [b for b, n in enumerate(CASES[name][7]) if n >= 64]
    assert rel_err(to_np_f32(got)[long], want[long]) <= 2e-2


@pytest.mark.parametrize("name", ["cut_merged_in_kernel", "cut_five_waves"])
def test_the_library_s_own_scratch(name):
    cfg, inp, d = _inputs(name)
    want = api.ss_msa_attention(*_args(d), cfg.gamma, inp["scale"])
    for _ in range(2):
        got = api.ss_msa_attention_static(*_args(d), cfg.gamma, inp["scale"], torch.full_like(d["q"], 3.0))
        assert torch.equal(got, want)


@pytest.mark.parametrize("name", ["cut_merged_in_kernel", "cut_eight_waves"])
def test_replays_cut_by_the_lengths_they_find(name):
    # one captured call, replayed on lengths that are cut anew, that fill the table's used part and that are empty
    cfg, inp, d = _inputs(name)
    shape, most = _shape(name), max(CASES[name][7])
    ws = api.ss_msa_workspace(*shape, DEV)
    out = torch.zeros_like(d["q"])
    call = lambda o, w: api.ss_msa_attention(*_args(d), cfg.gamma, inp["scale"], out=o, workspace=w)
    call(out, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(out, ws)
    B = shape[0]
    for lens in (CASES[name][7], [most] * B, [0] * B, [most // (i + 1) for i in range(B)], CASES[name][7]):
        d["seq_lens"].copy_(torch.tensor(lens, dtype=torch.int32))
        out.fill_(3.0)
        graph.replay()
        assert torch.equal(out, call(torch.full_like(out, 5.0), api.ss_msa_workspace(*shape, DEV))), lens


@pytest.mark.parametrize("room", [1.0, 1.1])
def test_batches_that_fill_the_table_keep_the_host_s_cut(room):
    # lengths of 7/8 of the capacity and more: looked at on the device, and the result is the forced host's cut's
    B, H, Hkv, D, page, T, gamma = 2, 12, 2, 64, 16, 32, 2
    CASES["even"] = (B, H, Hkv, D, page, T, gamma, [9000, 8900], room, False)
    try:
        cfg, inp, d = _inputs("even")
        where, n = api.ss_msa_plan_splits(*_shape("even"), [9000, 8900])
    finally:
        del CASES["even"]
    assert where == 1 and min(n) > 1
    got = api.ss_msa_attention(*_args(d), gamma, inp["scale"])
    a = [to_np_f32(inp[k]) for k in ("q", "k_new", "v_new", "k_cache", "v_cache")]
    want = oracle.msa_attention(*a, d["block_table"].cpu().numpy(), np.array([9000, 8900], np.int32), d["parent"].cpu().numpy(), gamma, inp["scale"])
    assert rel_err(to_np_f32(got), want) <= 2e-2


@pytest.mark.parametrize("lens,where", [([4100, 4200, 4300, 3000], 1), ([4300, 200, 4300, 3000], 2)])
def test_large_batches_of_nearly_full_sequences_keep_the_host_s_cut(lens, where):
    # 320 items: the work of the whole batch decides.  Against the kernel under two forced split lengths.  Either side
    # rounds probabilities and outputs to bf16, at most 2^-9 of each, and the values are random: the sums of the rounding
    # errors weigh no more against the result than they do term by term, 4 x 2^-9 of it in the 2-norm
    CASES["nearly_full"] = (4, 64, 16, 64, 16, 32, 4, lens, 4304 / max(lens), True)
    try:
        cfg, inp, d = _inputs("nearly_full")
        assert api.ss_msa_plan_splits(*_shape("nearly_full"), lens)[0] == where
    finally:
        del CASES["nearly_full"]
    got = api.ss_msa_attention(*_args(d), 4, inp["scale"])
    for keys in (1088, 2176):
        api.ss_msa_set_split_keys(keys)
        try:
            want = api.ss_msa_attention(*_args(d), 4, inp["scale"])
        finally:
            api.ss_msa_set_split_keys(0)
        g, w = got.float(), want.float()
        assert (g - w).norm() <= 2.0 ** -7 * w.norm()
