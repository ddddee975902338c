"""The fused tail where its loops and maxima can go wrong: more vocabulary tiles than lanes of a stream's waves, more rows
than waves, paths as deep as the tree, malformed parents, no streams, equal logits.  Against the oracle's verification and
drafting on the top-K that the stand-alone call finds (integers: exact)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2402_11131_amd import api, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = {
    # dtype, B, T, gamma, K, max_depth, draft branching, d, V, tree
    "tiles_beyond_the_lanes": (torch.bfloat16, 2, 40, 8, 3, 4, (3, 1, 1, 1, 1, 1, 1, 1), 64, 34000, "wide"),
    "tiles_twice_round": (torch.bfloat16, 1, 5, 1, 8, 2, (8,), 64, 66000, "wide"),
    "deep_chain": (torch.float32, 2, 64, 2, 2, 63, (2, 2), 32, 200, "chain"),
    "deeper_than_allowed": (torch.float32, 2, 30, 2, 2, 6, (2, 2), 32, 200, "chain"),
    "malformed_parents": (torch.bfloat16, 3, 33, 4, 4, 3, (4, 2, 1, 1), 64, 3000, "malformed"),
    "no_streams": (torch.bfloat16, 2, 17, 0, 1, 3, (), 64, 700, "wide"),
    "equal_logits": (torch.bfloat16, 2, 16, 4, 4, 3, (4, 2, 1, 1), 64, 5000, "equal"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_tail(name):
    dt, B, T, gamma, K, md, dbr, d, V, kind = CASES[name]
    R, rng = T * (1 + gamma), synth.rng_for(41)
    g = torch.Generator().manual_seed(7)
    W = torch.randn(V, d, generator=g)
    if kind == "equal":
        W = W[torch.arange(V) % 37]          # every logit comes 135 times, in all tiles
    hidden = torch.randn(B * R, d, generator=g)
    if kind == "chain":
        parent = np.tile(np.arange(-1, T - 1, dtype=np.int32), (B, 1))
    else:
        parent = synth.make_trees(5, B, T, (8, 4, 2), 3)
        if kind == "malformed":
            parent[:, 1::3], parent[0, 0] = rng.integers(-5, T + 5, parent[:, 1::3].shape), 9
    hidden, W = hidden.to(dt).to(DEV), W.to(dt).to(DEV)
    idx, _ = api.ss_lm_head_argmax_topk(hidden, W, K)
    top = idx.cpu().numpy().reshape(B, R, K)
    tok = rng.integers(0, V, (B, T)).astype(np.int32)
    for b in range(B):                       # most edges match; sequence 1 misses one in the middle
        for i in range(1, T):
            p = int(parent[b, i])
            p = p if 0 <= p < i else 0
            if rng.random() < 0.9 or kind == "chain":
                tok[b, i] = top[b, p, 0]
        if b == 1:
            tok[b, T // 2] = -1
    ver = oracle.tree_verify(tok, parent, np.ascontiguousarray(top[:, :T, 0]), md)
    out = api.ss_lm_head_verify_draft(hidden, W, K, torch.from_numpy(tok).to(DEV), torch.from_numpy(parent).to(DEV), gamma, md,
                                      **(dict(branching=dbr) if gamma else dict(tmpl_parent=torch.tensor([-1], dtype=torch.int32, device=DEV),
                                                                                tmpl_rank=torch.zeros(1, dtype=torch.int32, device=DEV))))
    for k in ("n_accept", "last", "bonus", "path", "out_tokens"):
        assert np.array_equal(out[k].cpu().numpy(), ver[k]), k
    assert np.array_equal(out["main_argmax"].cpu().numpy(), top[:, :T, 0])
    if kind == "chain":
        assert ver["n_accept"][0] == min(md, T - 1)
    if gamma:
        tp, tr, _ = oracle.full_tree_template(dbr)
        nxt, npar = oracle.tree_draft(np.ascontiguousarray(top[:, T:].reshape(B, T, gamma, K)), ver["last"], ver["bonus"], tp, tr)
        assert np.array_equal(out["next_tok"].cpu().numpy(), nxt) and np.array_equal(out["next_parent"].cpu().numpy(), npar)
    else:
        assert np.array_equal(out["next_tok"].cpu().numpy()[:, 0], ver["bonus"])
    # the stand-alone verification on the same inputs
    alone = api.ss_tree_verify(torch.from_numpy(tok).to(DEV), torch.from_numpy(parent).to(DEV), idx, md, batch_stride=R * K, node_stride=K)
    for k in ("n_accept", "last", "bonus", "path", "out_tokens"):
        assert torch.equal(alone[k], out[k]), k


@pytest.mark.parametrize("name", ["nan_rows", "few_numbers"])
def test_ranks_without_a_candidate(name):
    # A row with fewer than K logits that are numbers (its hidden state is NaN, or most of W is): the ranks that are left get
    # what the stand-alone top-K gives them, whatever a call before left behind.
    B, T, gamma, K, d, V, dbr = 3, 16, 4, 4, 64, 300, (4, 2, 1, 1)
    R = T * (1 + gamma)
    g = torch.Generator().manual_seed(11)
    hidden, W = torch.randn(B * R, d, generator=g), torch.randn(V, d, generator=g)
    parent = synth.make_trees(5, B, T, (4, 2, 2), 3)
    tok = synth.make_draft_tokens(6, parent, V)
    t_dev, p_dev = torch.from_numpy(tok).to(DEV), torch.from_numpy(parent).to(DEV)
    call = lambda h, w: api.ss_lm_head_verify_draft(h.to(DEV), w.to(DEV), K, t_dev, p_dev, gamma, 3, branching=dbr)
    call(hidden, W)                          # leaves tokens of its own where the next call's lists go
    if name == "nan_rows":
        hidden.view(B, R, d)[:, T + 1::2] = float("nan")      # every other stream row
        hidden.view(B, R, d)[2] = float("nan")                # all rows of a sequence, main rows too
    else:
        W[torch.arange(V) % 128 != 5] = float("nan")          # ids 5, 133 and 261: three numbers per row
    idx, _ = api.ss_lm_head_argmax_topk(hidden.to(DEV), W.to(DEV), K)
    ver = api.ss_tree_verify(t_dev, p_dev, idx, 3, batch_stride=R * K, node_stride=K)
    nxt, _ = api.ss_tree_draft(idx, K, ver["last"], ver["bonus"], T, gamma, branching=dbr, batch_stride=R * K, offset=T * K)
    assert int(nxt.max()) == np.iinfo(np.int32).max
    out = call(hidden, W)
    for k in ("n_accept", "last", "bonus", "path", "out_tokens"):
        assert torch.equal(out[k], ver[k]), k
    assert torch.equal(out["next_tok"], nxt)
