"""The work that users of this framework have it do, as cases that can be timed and compared.

Every case is one pass of a decode loop's own calls (paper_2402_11131_amd.api) on inputs that are already on the
GPU, enqueued on the current stream without a host synchronisation:

  step    one verify-and-speculate step: multi-stream attention of the last N_s layers, then LM head + verification +
          drafting.  The layers' own q/k/v and the last hidden states are inputs (the dense maps between them are the
          kind `layer`).
  layer   the dense maps of one layer on the step's rows: QKV, attention output, gate+up, down.
  entry   the way into the first multi-stream layer: the pruning layer on the main rows (log-sum-exp of the early-exit
          logits, transition probabilities, pruned trees), then stream insertion through the layer's QKV map.
  pruned  what follows it on pruned trees: the rows that were kept, attention and output map of the last N_s layers
          and the tail of the step on those rows only.
  commit  the end of a step: pages for the accepted tokens, then their keys / values into every layer's cache.

Sequences of a batch have lengths from l_min to l_max; `room` is the capacity of the block table over the longest
sequence (1: no page to spare; a serving loop keeps a table for the longest sequence it allows).
"""
import math

import numpy as np
import torch

from paper_2402_11131_amd import api, synth

DEVICE = "cuda:0"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
P_MATCH = 0.7  # an edge of the planted path is accepted with this probability, until the first miss


def listed():
    return [
        # The smallest step: one fp32 layer of 4 x 64 heads, 8-node tree, vocabulary 1000.  Launches and latency.
        dict(name="step_f32", kind="step", dtype="f32", b=1, h=4, hkv=4, d=64, l_min=128, l_max=128, room=1.0, t=8,
             gamma=3, depth=3, page=16, layers=1, vocab=1000, k=2),
        # The step right after a prompt: no draft yet, so the tree is its root and the streams make the first draft.
        dict(name="step_root", kind="step", dtype="bf16", b=2, h=32, hkv=32, d=64, l_min=411, l_max=777, room=4.0, t=1,
             gamma=4, depth=3, page=16, layers=4, vocab=32000, k=4),
        # One user, batch 1, as the paper measures: 32 x 128 heads, 2048 cached tokens, 16-node tree, 4 streams.
        dict(name="step_b1", kind="step", dtype="bf16", b=1, h=32, hkv=32, d=128, l_min=2048, l_max=2048, room=1.0, t=16,
             gamma=4, depth=3, page=16, layers=4, vocab=32000, k=4),
        # The headline step: 4 sequences of 4096 cached tokens.
        dict(name="step_b4", kind="step", dtype="bf16", b=4, h=32, hkv=32, d=128, l_min=4096, l_max=4096, room=1.0, t=16,
             gamma=4, depth=3, page=16, layers=4, vocab=32000, k=4),
        # Two sequences of uneven length with grouped query heads, ragged lengths, a table with room to grow.
        dict(name="step_gqa_b2", kind="step", dtype="bf16", b=2, h=32, hkv=8, d=128, l_min=3001, l_max=9005, room=1.8,
             t=24, gamma=3, depth=3, page=64, layers=4, vocab=32000, k=4),
        # Batched decode: the attention of 16 sequences of 1024 to 4096 cached tokens.
        dict(name="attn_b16", kind="step", dtype="bf16", b=16, h=32, hkv=32, d=128, l_min=1024, l_max=4096, room=1.0,
             t=16, gamma=4, depth=3, page=16, layers=4, vocab=0, k=4),
        # Long context: 8 sequences of 32768 cached tokens, grouped query heads, 160 rows each.
        dict(name="attn_gqa_32k", kind="step", dtype="bf16", b=8, h=32, hkv=8, d=128, l_min=32768, l_max=32768, room=1.0,
             t=32, gamma=4, depth=4, page=64, layers=1, vocab=0, k=4),
        # Dense maps of a layer on the rows of one sequence (80) and of four (320).
        dict(name="layer_b1", kind="layer", dtype="bf16", rows=80, d_model=4096, d_ff=11008, qkv=12288),
        dict(name="layer_b4", kind="layer", dtype="bf16", rows=320, d_model=4096, d_ff=11008, qkv=12288),
        # Into the first multi-stream layer with four sequences of 16 nodes.
        dict(name="entry_b4", kind="entry", dtype="bf16", b=4, t=16, gamma=4, depth=3, d_model=4096, vocab=32000, qkv=12288),
        # Grouped query heads after pruning: 8 sequences, from a third to two thirds of every tree kept.
        dict(name="pruned_b8", kind="pruned", dtype="bf16", b=8, h=32, hkv=8, d=128, l_min=2000, l_max=8192, room=1.0, t=32,
             gamma=4, depth=4, page=64, layers=2, vocab=32000, k=4, keep=0.5),
        # The accepted tokens of 16 sequences into the caches of four layers.
        dict(name="commit_b16", kind="commit", dtype="bf16", b=16, h=32, hkv=32, d=128, l_min=101, l_max=509, room=1.1,
             t=16, gamma=4, depth=4, page=16, layers=4),
    ]


# ------------------------------------------------------------------ more cases of the same ranges

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choice(["step", "step", "step", "step_f32", "step_f32", "attn", "attn", "layer", "layer", "entry", "pruned", "commit"])
    tree = dict(t=rng.randint(1, 32), gamma=rng.randint(2, 5))
    tree["depth"] = min(tree["gamma"], rng.randint(2, 4))
    h, hkv, d = rng.choice([(32, 32, 128), (32, 8, 128), (32, 32, 64), (32, 4, 128), (16, 16, 128), (40, 8, 64)])
    heads = dict(h=h, hkv=hkv, d=d)
    longest = _log_int(rng, 64, 8192)
    cache = dict(l_min=rng.randint(longest // 3, longest), l_max=longest, room=rng.choice([1.0, 1.0, 1.5, 2.0, 4.0]),
                 page=rng.choice([16, 16, 32, 64]))
    k = rng.choice([1, 2, 4, 8])
    if kind == "step_f32":
        h = rng.choice([4, 8])
        cache.update(l_max=min(longest, 1024), l_min=min(cache["l_min"], 1024))
        return dict(kind="step", dtype="f32", b=rng.randint(1, 4), h=h, hkv=h, d=64, layers=rng.randint(1, 2),
                    vocab=_log_int(rng, 500, 8000), k=k, **cache, **tree)
    if kind == "step":
        return dict(kind="step", dtype="bf16", b=_log_int(rng, 1, 8), layers=rng.randint(1, 4), vocab=_log_int(rng, 2000, 50000),
                    k=k, **heads, **cache, **tree)
    if kind == "attn":
        longest = _log_int(rng, 256, 32768)
        cache.update(l_max=longest, l_min=rng.randint(longest // 3, longest))
        return dict(kind="step", dtype="bf16", b=_log_int(rng, 1, 16), layers=rng.randint(1, 4), vocab=0, k=4, **heads, **cache, **tree)
    if kind == "layer":
        d_model = rng.choice([2048, 3072, 4096, 5120])
        return dict(kind="layer", dtype="bf16", rows=_log_int(rng, 5, 640), d_model=d_model, d_ff=64 * rng.randint(80, 216),
                    qkv=rng.choice([d_model * 3, d_model + d_model // 2]))
    if kind == "entry":
        d_model = rng.choice([2048, 4096])
        return dict(kind="entry", dtype="bf16", b=_log_int(rng, 1, 16), d_model=d_model, vocab=_log_int(rng, 2000, 50000),
                    qkv=d_model * 3, **tree)
    if kind == "pruned":
        tree["t"] = max(tree["t"], 8)
        return dict(kind="pruned", dtype="bf16", b=_log_int(rng, 1, 8), layers=rng.randint(1, 3), vocab=_log_int(rng, 2000, 50000),
                    k=k, keep=rng.uniform(0.3, 0.8), **heads, **cache, **tree)
    tree["t"] = max(tree["t"], 2)
    return dict(kind="commit", dtype="bf16", b=_log_int(rng, 1, 16), layers=rng.randint(1, 4), **heads,
                **dict(cache, l_max=min(longest, 1024), l_min=min(cache["l_min"], 1024), room=max(cache["room"], 1.5)), **tree)


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 4e12, w["flops"] / (1e15 if case["dtype"] == "bf16" else 2e13))


def draw(rng):
    most = 0.8 * max(_cost(c) for c in listed())
    while True:
        case = _draw_once(rng)
        if _cost(case) <= most:
            return case


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _normal(gen, shape, dtype, std=1.0):
    return torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32).mul_(std).to(dtype)


def _lengths(case, seed=None):
    """The batch's lengths, evenly from l_min to l_max; in an order of the seed's."""
    lens = np.rint(np.linspace(case["l_max"], case["l_min"], case["b"])).astype(np.int32)
    return lens if seed is None else synth.rng_for(seed ^ 0x5EED).permutation(lens)


def _capacity(case):
    """Tokens a row of the block table has entries for."""
    return -(-int(math.ceil(case["l_max"] * case["room"])) // case["page"]) * case["page"]


def _table(case, seed, lens):
    """Pages of all sequences in a pool with a quarter to spare; entries past a sequence's pages are unused."""
    used, num_pages = synth.make_page_table(seed, lens, case["page"])
    table = np.zeros((case["b"], _capacity(case) // case["page"]), np.int32)
    table[:, :used.shape[1]] = used
    return table, num_pages


def _widths(case):
    """Children per node at each depth: what k-wide streams allow at most, wide enough for t nodes."""
    return (8,) * case["depth"]


def _branching(case):
    """The next tree's shape: k children of the root, fewer below."""
    k, out = case["k"], [case["k"]]
    for _ in range(case["gamma"] - 1):
        out.append(2 if k in (2, 4) and len(out) == 1 else 1)
    return tuple(out)


def _trees(case, seed):
    return synth.make_trees(seed ^ 0x7EE, case["b"], case["t"], _widths(case), case["depth"])


def _layer_inputs(case, gen, num_pages):
    dt = DTYPES[case["dtype"]]
    b, r, h, hkv, d, page = case["b"], case["t"] * (1 + case["gamma"]), case["h"], case["hkv"], case["d"], case["page"]
    return dict(q=_normal(gen, (b, r, h, d), dt), k_new=_normal(gen, (b, r, hkv, d), dt), v_new=_normal(gen, (b, r, hkv, d), dt),
                k_cache=_normal(gen, (num_pages, hkv, page, d), dt), v_cache=_normal(gen, (num_pages, hkv, d, page), dt),
                out=torch.zeros(b, r, h, d, dtype=dt, device=DEVICE))


def _attention_state(case, seed, gen):
    lens = _lengths(case, seed)
    table, num_pages = _table(case, seed, lens)
    code = api.SS_F32 if case["dtype"] == "f32" else api.SS_BF16
    return dict(layers=[_layer_inputs(case, gen, num_pages) for _ in range(case["layers"])],
                table=torch.from_numpy(table).to(DEVICE), lens=torch.from_numpy(lens).to(DEVICE),
                scale=1.0 / math.sqrt(case["d"]),
                ws=api.ss_msa_workspace(case["b"], case["t"], case["gamma"], case["h"], case["hkv"], case["d"],
                                        _capacity(case), code, DEVICE))


def _head_state(case, seed, gen, parent, tok):
    """Last hidden states, LM head and draft tokens, with the path that the main stream will accept planted."""
    dt = DTYPES[case["dtype"]]
    n, d_model = case["b"] * case["t"] * (1 + case["gamma"]), case["h"] * case["d"]
    hidden, W = _normal(gen, (n, d_model), dt), _normal(gen, (case["vocab"], d_model), dt, 0.02)
    synth.plant_acceptance(seed, parent, tok, hidden, W, case["t"] * (1 + case["gamma"]), P_MATCH)
    code = api.SS_F32 if case["dtype"] == "f32" else api.SS_BF16
    need = api.ss_lm_head_workspace_bytes(n, d_model, case["vocab"], case["k"], code)
    return dict(hidden=hidden, W=W, lm_ws=torch.empty(need, dtype=torch.uint8, device=DEVICE))


def _prepare_step(case, seed):
    gen = _gen(seed)
    s = _attention_state(case, seed, gen)
    parent = _trees(case, seed)
    s["parent"] = torch.from_numpy(parent).to(DEVICE)
    if case["vocab"]:
        tok = synth.make_draft_tokens(seed, parent, case["vocab"])
        s.update(_head_state(case, seed, gen, parent, tok), tok=torch.from_numpy(tok).to(DEVICE))
    return s


def _run_step(case, s):
    outs = [api.ss_msa_attention(x["q"], x["k_new"], x["v_new"], x["k_cache"], x["v_cache"], s["table"], s["lens"], s["parent"],
                                 case["gamma"], s["scale"], out=x["out"], workspace=s["ws"]) for x in s["layers"]]
    if not case["vocab"]:
        return outs
    s["tail"] = api.ss_lm_head_verify_draft(s["hidden"], s["W"], case["k"], s["tok"], s["parent"], case["gamma"], case["depth"],
                                            branching=_branching(case), workspace=s["lm_ws"], out=s.get("tail"))
    return outs, s["tail"]


def _maps(case):
    return dict(qkv=(case["d_model"], case["qkv"]), out=(case["d_model"], case["d_model"]),
                gate_up=(case["d_model"], 2 * case["d_ff"]), down=(case["d_ff"], case["d_model"]))


def _prepare_layer(case, seed):
    gen, dt, n, s = _gen(seed), DTYPES[case["dtype"]], case["rows"], []
    need = 1
    for d_in, d_out in _maps(case).values():
        s.append(dict(x=_normal(gen, (n, d_in), dt), W=_normal(gen, (d_out, d_in), dt, 0.02),
                      y=torch.empty(n, d_out, dtype=dt, device=DEVICE)))
        need = max(need, api.ss_linear_rows_workspace_bytes(n, d_in, d_out, api.SS_BF16))
    return dict(maps=s, ws=torch.empty(need, dtype=torch.uint8, device=DEVICE))


def _run_layer(case, s):
    return [api.ss_linear_rows_ws(m["x"], m["W"], m["y"], workspace=s["ws"]) for m in s["maps"]]


def _prepare_entry(case, seed):
    gen, dt = _gen(seed), DTYPES[case["dtype"]]
    b, t, gamma, d_model = case["b"], case["t"], case["gamma"], case["d_model"]
    parent = _trees(case, seed)
    tok = synth.make_draft_tokens(seed, parent, case["vocab"])
    exit_h, W = _normal(gen, (b * t, d_model), dt), _normal(gen, (case["vocab"], d_model), dt, 0.02)
    # every second node is one that its parent expects
    kids = [(i * t + int(parent[i, c]), int(tok[i, c])) for i in range(b) for c in range(1, t, 2)]
    if kids:
        rows, toks = (torch.tensor(v, device=DEVICE) for v in zip(*kids))
        to_parent = (rows == torch.arange(b * t, device=DEVICE)[:, None]).float() * (12.0 / (0.02 * math.sqrt(d_model)))
        exit_h = (exit_h.float() + to_parent @ W[toks].float()).to(dt)
    ws = api.ss_lm_head_workspace_bytes(b * t, d_model, case["vocab"], 1, api.SS_BF16)
    ins = api.load_library().ss_stream_insert_linear_workspace_bytes(b, t, gamma, d_model, case["qkv"], api.SS_BF16, 0)
    return dict(exit_h=exit_h, W=W, M=_normal(gen, (b, t, d_model), dt), P=_normal(gen, (gamma, d_model), dt),
                Wqkv=_normal(gen, (case["qkv"], d_model), dt, 0.02), tok=torch.from_numpy(tok).to(DEVICE),
                parent=torch.from_numpy(parent).to(DEVICE), lse=torch.empty(b * t, dtype=torch.float32, device=DEVICE),
                prob=torch.empty(b, t, dtype=torch.float32, device=DEVICE),
                Y=torch.empty(b, t * (1 + gamma), case["qkv"], dtype=dt, device=DEVICE),
                ws=torch.empty(ws, dtype=torch.uint8, device=DEVICE), ins_ws=torch.empty(ins, dtype=torch.uint8, device=DEVICE))


def _run_entry(case, s):
    api.ss_lm_head_logsumexp(s["exit_h"], s["W"], lse=s["lse"], workspace=s["ws"])
    api.ss_transition_probs(s["exit_h"].view(case["b"], case["t"], case["d_model"]), s["W"], s["tok"], s["parent"], s["lse"], prob=s["prob"])
    trees = api.ss_tree_prune(s["tok"], s["parent"], s["prob"], 0.05)
    Y = api.ss_stream_insert_linear(s["M"], s["P"], s["Wqkv"], Y=s["Y"], workspace=s["ins_ws"])
    return s["lse"], s["prob"], trees, Y


def _kept(case):
    """Nodes kept of each tree: around keep * t, from two thirds to four thirds of it over the batch."""
    b, t = case["b"], case["t"]
    return [min(t, max(1, round(case["keep"] * t * (2 + (2 * i / (b - 1) if b > 1 else 1)) / 3))) for i in range(b)]


def _prepare_pruned(case, seed):
    gen, dt, rng = _gen(seed), DTYPES[case["dtype"]], synth.rng_for(seed ^ 0x9A11)
    s = _attention_state(case, seed, gen)
    b, t, r, d_model = case["b"], case["t"], case["t"] * (1 + case["gamma"]), case["h"] * case["d"]
    parent = _trees(case, seed)
    tok = synth.make_draft_tokens(seed, parent, case["vocab"])
    prob = np.full((b, t), 0.01, np.float32)
    for i, n in enumerate(_kept(case)):  # a random sub-tree of n nodes is likely
        kept = {0}
        while len(kept) < n:
            kept.add(int(rng.choice([c for c in range(1, t) if c not in kept and int(parent[i, c]) in kept])))
        prob[i, sorted(kept)] = rng.uniform(0.06, 1.0, n)
    s.update(tok=torch.from_numpy(tok).to(DEVICE), parent=torch.from_numpy(parent).to(DEVICE), prob=torch.from_numpy(prob).to(DEVICE))
    # the path to accept is planted in the numbering the trees have after pruning
    trees = api.ss_tree_prune(s["tok"], s["parent"], s["prob"], 0.05)
    small, small_tok, n_nodes = (trees[k].cpu().numpy() for k in ("parent", "tok", "n_nodes"))
    hidden, W = _normal(gen, (b * r, d_model), dt), _normal(gen, (case["vocab"], d_model), dt, 0.02)
    for i in range(b):
        hold = hidden[i * r:(i + 1) * r]
        n = int(n_nodes[i])
        synth.plant_acceptance(seed + i, small[i:i + 1, :n], small_tok[i:i + 1, :n], hold, W, r, P_MATCH)
    for x in s["layers"]:
        x.update(Wo=_normal(gen, (d_model, d_model), dt, 0.02), y=torch.zeros(b * r, d_model, dtype=dt, device=DEVICE))
    need = api.ss_lm_head_workspace_bytes(b * r, d_model, case["vocab"], case["k"], api.SS_BF16)
    s.update(hidden=hidden, W=W, lm_ws=torch.empty(need, dtype=torch.uint8, device=DEVICE),
             live=(torch.zeros(b * r, dtype=torch.int32, device=DEVICE), torch.zeros(1, dtype=torch.int32, device=DEVICE)),
             plan=max(1, int(case["keep"] * b * r)))
    return s


def _run_pruned(case, s):
    b, r, d_model = case["b"], case["t"] * (1 + case["gamma"]), case["h"] * case["d"]
    trees = api.ss_tree_prune(s["tok"], s["parent"], s["prob"], 0.05)
    live = api.ss_live_rows(trees["n_nodes"], case["t"], case["gamma"], *s["live"])
    for x in s["layers"]:
        api.ss_msa_attention(x["q"], x["k_new"], x["v_new"], x["k_cache"], x["v_cache"], s["table"], s["lens"], trees["parent"],
                             case["gamma"], s["scale"], out=x["out"], workspace=s["ws"], n_nodes=trees["n_nodes"])
        api.ss_linear_rows(x["out"].view(b * r, d_model), x["Wo"], x["y"], live=live, plan_rows=s["plan"])
    s["tail"] = api.ss_lm_head_verify_draft(s["hidden"], s["W"], case["k"], trees["tok"], trees["parent"], case["gamma"],
                                            case["depth"], branching=_branching(case), workspace=s["lm_ws"], out=s.get("tail"),
                                            live=live, plan_rows=s["plan"])
    # the arg-max of rows that pruning removed is not defined
    tail = {k: v for k, v in s["tail"].items() if k != "main_argmax"}
    return [(x["out"], x["y"]) for x in s["layers"]], trees["n_nodes"], tail


def _accepted(case):
    """Accepted tokens of each sequence: every number from none to the depth, but no more than the tree has."""
    return np.array([i % (min(case["depth"], case["t"] - 1) + 1) for i in range(case["b"])], np.int32)


def _prepare_commit(case, seed):
    gen, rng = _gen(seed), synth.rng_for(seed ^ 0xC033)
    s = _attention_state(case, seed, gen)
    lens, acc, depth = _lengths(case, seed), _accepted(case), case["depth"]
    path = np.full((case["b"], depth + 1), -1, np.int32)
    for i, n in enumerate(acc):
        path[i, :n + 1] = np.concatenate([[0], 1 + np.sort(rng.permutation(case["t"] - 1)[:n])])
    num_pages = s["layers"][0]["k_cache"].shape[0]
    table = s["table"].cpu().numpy()
    used = {int(table[i, p]) for i, n in enumerate(lens) for p in range(-(-int(n) // case["page"]))}
    spare = [p for p in range(num_pages) if p not in used]
    # every sequence grows by at most two pages; a pool without that many spare pages gets them
    extra = max(0, 2 * case["b"] - len(spare))
    if extra:
        for x in s["layers"]:
            for name in ("k_cache", "v_cache"):
                shape = list(x[name].shape)
                x[name] = torch.cat([x[name], _normal(gen, [extra] + shape[1:], x[name].dtype)])
    spare += range(num_pages, num_pages + extra)
    s.update(path=torch.from_numpy(path).to(DEVICE), acc=torch.from_numpy(acc).to(DEVICE),
             free=torch.tensor(rng.permutation(spare).astype(np.int32), device=DEVICE), n_free=len(spare),
             free_count=torch.zeros(1, dtype=torch.int32, device=DEVICE), n_commit=torch.zeros_like(s["lens"]),
             new_lens=torch.zeros_like(s["lens"]))
    return s


def _run_commit(case, s):
    s["free_count"].fill_(s["n_free"])  # pages of sequences that ended are back on the stack
    n = api.ss_kv_alloc_pages(s["table"], s["lens"], s["acc"], case["page"], case["depth"], s["free"], s["free_count"], n_commit=s["n_commit"])
    for x in s["layers"]:
        api.ss_kv_commit(x["k_new"], x["v_new"], x["k_cache"], x["v_cache"], s["table"], s["lens"], s["path"], n, case["gamma"],
                         new_seq_lens=s["new_lens"])
    return [(x["k_cache"], x["v_cache"]) for x in s["layers"]], s["table"], s["free_count"], n, s["new_lens"]


_KINDS = dict(step=(_prepare_step, _run_step), layer=(_prepare_layer, _run_layer), entry=(_prepare_entry, _run_entry),
              pruned=(_prepare_pruned, _run_pruned), commit=(_prepare_commit, _run_commit))


def prepare(case, seed):
    return case, _KINDS[case["kind"]][0](case, seed)


def run(state):
    case, s = state
    return _KINDS[case["kind"]][1](case, s)


# ------------------------------------------------------------------ what a pass cannot do without

def _add(*parts):
    return {k: float(sum(p[k] for p in parts)) for k in ("bytes", "flops")}


def _attention_work(case, rows):
    """Attention of one layer: the caches once, new keys / values, q and out of the computed rows."""
    e = 2 if case["dtype"] == "bf16" else 4
    lens = [int(n) for n in _lengths(case)]
    kv = sum(2 * (n + r) * case["hkv"] * case["d"] * e for n, r in zip(lens, rows))
    return {"bytes": kv + 2 * sum(rows) * case["h"] * case["d"] * e + 4 * sum(n // case["page"] for n in lens),
            "flops": sum(4 * r * (n + r) * case["h"] * case["d"] for n, r in zip(lens, rows))}


def _map_work(n, d, v, e, out_bytes=None):
    return {"bytes": (n * d + v * d) * e + (n * v * e if out_bytes is None else out_bytes), "flops": 2 * n * d * v}


def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "layer":
        return _add(*[_map_work(case["rows"], d, v, e) for d, v in _maps(case).values()])
    if case["kind"] == "entry":
        n, d = case["b"] * case["t"], case["d_model"]
        y = n * (1 + case["gamma"]) * case["qkv"] * e
        return _add(_map_work(n, d, case["vocab"], e, 40 * n), _map_work(n + case["gamma"], d, case["qkv"], e, y))
    if case["kind"] == "commit":
        tokens = int(_accepted(case).sum()) + case["b"]
        return {"bytes": float(4 * tokens * case["layers"] * case["hkv"] * case["d"] * e + 24 * case["b"]), "flops": 0.0}
    kept = _kept(case) if case["kind"] == "pruned" else [case["t"]] * case["b"]
    rows = [n * (1 + case["gamma"]) for n in kept]
    parts = [_attention_work(case, rows)] * case["layers"]
    d_model = case["h"] * case["d"]
    if case["kind"] == "pruned":
        parts = parts + [_map_work(sum(rows), d_model, d_model, e)] * case["layers"]
    if case["vocab"]:
        parts = parts + [_map_work(sum(rows), d_model, case["vocab"], e, 64 * sum(kept))]
    return _add(*parts)


def tolerance(case):
    """About four times what the path differs by from the same sums in 64 bits: bf16 attention 2.3e-3 (largest element
    1.3e-2), dense maps 1.7e-3 (the rounding of the result); fp32 attention 3e-7 (1.6e-6).  Whole numbers are tokens,
    which may differ where two logits tie."""
    if case["kind"] == "commit":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 2e-5, "differ": 0.002}
    return {"rel": 1e-2, "max": 6e-2, "differ": 0.002}


# ------------------------------------------------------------------ the same results from plain torch in 64 bits

def _clamped(parent):
    return [-1] + [p if 0 <= p < i else 0 for i, p in enumerate(parent) if i > 0]


def _sees(parent, gamma):
    """Which of a sequence's new rows each of them sees: a main row its ancestors and itself, a stream row those and the
    node's streams up to its own."""
    t = len(parent)
    up = torch.zeros(t, t, dtype=torch.bool)
    for i, p in enumerate(_clamped(parent)):
        if p >= 0:
            up[i] = up[p]
        up[i, i] = True
    see = torch.zeros(t * (1 + gamma), t * (1 + gamma), dtype=torch.bool)
    see[:t, :t] = up
    for i in range(t):
        for j in range(gamma):
            see[t + i * gamma + j, :t] = up[i]
            see[t + i * gamma + j, t + i * gamma:t + i * gamma + j + 1] = True
    return see.to(DEVICE)


def _exact_attention(case, s, x, trees):
    """Attention of one layer; trees: (parents, rows that count) of every sequence."""
    out = torch.zeros_like(x["out"], dtype=torch.float64)
    table, lens, page, g = s["table"].cpu(), s["lens"].cpu(), case["page"], case["h"] // case["hkv"]
    for i, (parent, rows) in enumerate(trees):
        n = int(lens[i])
        pages, see = table[i, :-(-n // page)].long().to(DEVICE), _sees(parent, case["gamma"])[rows]
        for j in range(case["hkv"]):
            k = torch.cat([x["k_cache"][pages, j].reshape(-1, case["d"])[:n], x["k_new"][i, :, j]]).double()
            v = torch.cat([x["v_cache"][pages, j].transpose(1, 2).reshape(-1, case["d"])[:n], x["v_new"][i, :, j]]).double()
            for h in range(j * g, (j + 1) * g):
                score = (x["q"][i, rows, h].double() @ k.T) * s["scale"]
                score[:, n:].masked_fill_(~see, -math.inf)
                out[i, rows, h] = torch.softmax(score, 1) @ v
    return out


def _product(x, W):
    """x . W^T, a slice of W at a time."""
    return torch.cat([x.double() @ w.double().T for w in W.split(4096)], 1)


_TAIL = ("n_accept", "last", "bonus", "path", "out_tokens", "next_tok", "next_parent")


def _exact_step(case, s):
    trees = [(p, slice(None)) for p in s["parent"].cpu().tolist()]
    outs = [_exact_attention(case, s, x, trees) for x in s["layers"]]
    return (outs, dict.fromkeys(_TAIL + ("main_argmax",))) if case["vocab"] else outs


def _exact_layer(case, s):
    return [_product(m["x"], m["W"]) for m in s["maps"]]


def _exact_entry(case, s):
    b, t, gamma = case["b"], case["t"], case["gamma"]
    logits = _product(s["exit_h"], s["W"])
    lse = torch.logsumexp(logits, 1)
    parent, tok = s["parent"].cpu().tolist(), s["tok"].cpu().tolist()
    prob = torch.ones(b, t, dtype=torch.float64, device=DEVICE)
    for i in range(b):
        for c, p in enumerate(_clamped(parent[i])):
            if c:
                prob[i, c] = torch.exp(logits[i * t + p, tok[i][c]] - lse[i * t + p])
    m, p = _product(s["M"].view(b * t, -1), s["Wqkv"]).view(b, t, -1), _product(s["P"], s["Wqkv"])
    streams = (m[:, :, None] + p).view(b, t * gamma, -1)
    return lse, prob, dict.fromkeys(("keep", "tok", "parent", "old_index", "n_nodes")), torch.cat([m, streams], 1)


def _exact_pruned(case, s):
    t, gamma, trees, live = case["t"], case["gamma"], [], []
    for i, (parent, prob) in enumerate(zip(s["parent"].cpu().tolist(), s["prob"].cpu().tolist())):
        new, old = {}, _clamped(parent)
        for c in range(t):
            if c == 0 or (old[c] in new and prob[c] >= 0.05):
                new[c] = len(new)
        n = len(new)
        rows = list(range(n)) + list(range(t, t + n * gamma))
        trees.append(([new.get(old[c], -1) for c in new] + [0] * (t - n), torch.tensor(rows, device=DEVICE)))
        live += [i * t * (1 + gamma) + r for r in rows]
    layers = []
    for x in s["layers"]:
        out, y = _exact_attention(case, s, x, trees), torch.zeros_like(x["y"], dtype=torch.float64)
        y[live] = _product(out.view(len(y), -1)[live], x["Wo"])
        layers.append((out, y))
    return layers, None, dict.fromkeys(_TAIL)


def exact(case, seed):
    """The outputs that are computed numbers; tokens, trees and copied bytes have no such value."""
    if case["kind"] == "commit":
        return None
    kinds = dict(step=_exact_step, layer=_exact_layer, entry=_exact_entry, pruned=_exact_pruned)
    return kinds[case["kind"]](case, prepare(case, seed)[1])
