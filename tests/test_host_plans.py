"""Host logic of the launch plans (no GPU): how shapes are cut into splits, slices and workspaces."""
import ctypes

from paper_2402_11131_amd import api, synth


def _msa_plan(cfg, max_len):
    return api.ss_msa_plan(cfg.B, cfg.T, cfg.gamma, cfg.H, cfg.Hkv, cfg.D, max_len, api.SS_BF16 if cfg.dtype == "bf16" else api.SS_F32)


def test_attention_plans_of_the_five_workloads():
    c = synth.CONFIGS
    assert _msa_plan(c["c4"], 4096) == (2, 1)        # two splits, merged inside the attention kernel
    assert _msa_plan(c["c3"], 4096) == (1, 1)        # 512 (sequence, head) items: unsplit
    assert _msa_plan(c["c5"], 32768) == (4, 2)       # five row chunks of 128 rows x 64 KV heads x 4 splits = 5 whole rounds
    splits, kernels = _msa_plan(c["c2"], 2048)
    assert splits == 8 and kernels == 2              # one sequence: 8 splits and the merge kernel
    assert _msa_plan(c["c1"], 128)[1] in (1, 2)


def test_attention_workspace_grows_with_the_splits_and_holds_the_counters():
    c4 = synth.CONFIGS["c4"]
    lib = api.load_library()
    need = lib.ss_msa_workspace_bytes(c4.B, c4.T, c4.gamma, c4.H, c4.Hkv, c4.D, 4096, api.SS_BF16)
    partial_rows = c4.B * c4.H * 2 * c4.R                      # two splits
    assert need >= partial_rows * (c4.D + 1) * 4 + c4.B * c4.Hkv * 8 * 4
    assert lib.ss_msa_workspace_bytes(16, c4.T, c4.gamma, c4.H, c4.Hkv, c4.D, 4096, api.SS_BF16) <= 512   # c3: unsplit
    api.ss_msa_set_split_keys(1024)
    try:
        assert _msa_plan(c4, 4096) == (4, 2)                   # override: four splits go through the merge kernel
    finally:
        api.ss_msa_set_split_keys(0)
    assert _msa_plan(c4, 4096) == (2, 1)


def test_merge_in_the_kernel_stops_where_its_counters_fill_their_region():
    api.ss_msa_set_split_keys(1024)
    try:
        assert api.ss_msa_plan(256, 16, 4, 32, 32, 128, 2048, api.SS_BF16) == (2, 1)      # 8192 items
        assert api.ss_msa_plan(257, 16, 4, 32, 32, 128, 2048, api.SS_BF16) == (2, 2)      # 8224: the merge kernel
    finally:
        api.ss_msa_set_split_keys(0)


def test_projection_slices():
    bf, f32 = api.SS_BF16, api.SS_F32
    assert api.ss_linear_rows_splits(320, 11008, 4096, bf) == 4     # down map: few outputs, many features
    assert api.ss_linear_rows_splits(320, 4096, 4096, bf) == 4      # output map
    for V in (12288, 22016, 32000):                                 # QKV, gate+up, LM-head-sized: many outputs
        assert api.ss_linear_rows_splits(320, 4096, V, bf) == 1
    assert api.ss_linear_rows_splits(320, 11008, 4096, f32) == 1    # the fp32 kernel is never cut
    assert api.ss_linear_rows_splits(64, 192, 4096, bf) == 1        # three feature blocks cannot be cut in two or four
    assert api.ss_linear_rows_splits(0, 4096, 4096, bf) == 1
    assert api.ss_linear_rows_splits(320, 100, 4096, bf) == 0       # d % 64 != 0: refused, message set
    assert b"64" in api.load_library().ss_last_error()


def test_projection_workspace_matches_the_slices():
    bf = api.SS_BF16
    for N, d, V in ((320, 11008, 4096), (320, 4096, 4096), (96, 2048, 250), (320, 4096, 12288), (1, 64, 8)):
        s = api.ss_linear_rows_splits(N, d, V, bf)
        need = api.ss_linear_rows_workspace_bytes(N, d, V, bf)
        assert need == (s * N * V * 4 + 256 if s > 1 else 256)
    lib = api.load_library()
    one = ctypes.c_void_p(256)  # never dereferenced: validation fails first
    assert lib.ss_linear_rows_ws(one, one, 320, 11008, 4096, bf, one, one, 1024, None) == 4      # SS_ERR_WORKSPACE
    assert b"workspace" in lib.ss_last_error()
    assert lib.ss_linear_rows_ws(one, one, 320, 11008, 4096, bf, one, None, 0, None) == 4
    assert lib.ss_linear_rows_ws(None, one, 320, 11008, 4096, bf, one, one, 1 << 30, None) == 1  # SS_ERR_INVALID_ARG


def test_attention_refuses_a_cache_beyond_its_page_offsets():
    # bf16 path: page offsets are kept in units of 256 bytes in 32 bits, i.e. up to 1 TiB per cache tensor; the
    # check runs on the host before anything is enqueued (the pointers are never dereferenced)
    lib = api.load_library()
    one = ctypes.c_void_p(256)
    pages = (1 << 40) // (32 * 64 * 128 * 2) + 1
    rc = lib.ss_msa_attention(one, one, one, one, one, one, 4, pages, one, one, 1, 4, 1, 32, 32, 128, 64, 0.1,
                              api.SS_BF16, 0, one, None, 0, None)
    assert rc == 2 and b"1 TiB" in lib.ss_last_error()   # SS_ERR_UNSUPPORTED


# Batches that the device cuts: (B, T, gamma, H, Hkv, D, capacity, lengths, kept nodes or None)
_CUT_BATCHES = [
    (8, 32, 4, 32, 8, 128, 8192, [8192, 0, 0, 5000, 2500, 0, 7000, 4097], None),
    (8, 32, 4, 32, 8, 128, 8192, [0, 5299, 2500, 8192, 3993, 2500, 5000, 2500], [11, 32, 1, 20, 13, 8, 32, 2]),
    (8, 32, 4, 32, 8, 128, 8192, [0] * 8, None),
    (2, 24, 3, 32, 8, 128, 16256, [9005, 3001], None),
    (4, 16, 2, 48, 16, 64, 4096, [1100, 513, 0, 700], None),       # at most two splits each: merged in the attention kernel
    (64, 8, 2, 4, 1, 64, 8192, [(i * 37) % 600 for i in range(64)], None),
]


def _check_cuts():
    rng = synth.rng_for(7)
    for B, T, gamma, H, Hkv, D, cap, lens, kept in _CUT_BATCHES:
        most, _ = api.ss_msa_plan(B, T, gamma, H, Hkv, D, cap, api.SS_BF16)
        draws = [(lens, kept)]
        for _ in range(200):
            draws.append(([int(x) for x in rng.integers(0, cap + 1, B) * rng.integers(0, 2, B)],
                          None if rng.integers(0, 2) else [int(x) for x in rng.integers(1, T + 1, B)]))
        for lens, kept in draws:
            where, n = api.ss_msa_plan_splits(B, T, gamma, H, Hkv, D, cap, api.SS_BF16, lens, kept)
            assert where in (1, 2)
            assert all(k >= 1 for k in n), (lens, kept, n)                      # every sequence has a split 0
            assert sum(n) <= B * most, (lens, kept, n)                          # the workspace holds that many
            assert most != 2 or max(n) <= 2, (lens, kept, n)


def test_cut_of_an_uneven_batch_fits_the_workspace():
    import os
    import subprocess
    import sys
    _check_cuts()
    # the same for every kind of value SS_MSA_SPLIT0_EXTRA takes (read once per process): below -5 the step's own 160
    # rows count for nothing
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    code = "import sys; sys.path[:0] = [%r, %r]; import test_host_plans as t; t._check_cuts()" % (root, os.path.join(root, "tests"))
    for extra in (-64, -5, -4, 0, 64):
        r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, SS_MSA_SPLIT0_EXTRA=str(extra)), cwd=root,
                           stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
        assert r.returncode == 0, (extra, r.stdout[-2000:])


def _cut_by_hand(B, T, gamma, H, Hkv, n_slots, chunk_rows, groups, lens, n=None):
    """Cost of a cut by its own rule, rounds of the busiest XCD (workgroups are dealt to eight XCDs in turn, 32 at a
    time) x (blocks of the longest split + 4): of the cut n, or the least of all split lengths."""
    new = -(-T * (1 + gamma) // 32) + 2
    load = [-(-x // 32) + new for x in lens]
    chunks = -(-(H // Hkv) * T * (1 + gamma) // chunk_rows)

    def cost(c, n):
        return -(-(-(-sum(n) * Hkv // 8) * chunks) // 32) * (c + 4)
    if n is not None:
        return cost(max(-(-(-(-x // k)) // groups) * groups for x, k in zip(load, n)), n)
    cuts = [(c, [-(-x // c) for x in load]) for c in range(8, max(load) + groups, groups)]
    return min(cost(c, n) for c, n in cuts if sum(n) <= n_slots)


def test_cut_counts_the_workgroups_of_the_busiest_xcd():
    # four KV heads: the pieces of two sequences share the rounds of the eight XCDs
    rng = synth.rng_for(11)
    for B, T, gamma, H, Hkv, cap, chunk_rows, groups in ((2, 24, 3, 32, 4, 16256, 128, 2), (3, 24, 3, 32, 4, 16256, 128, 2),
                                                         (5, 8, 3, 24, 4, 16384, 64, 3), (2, 24, 3, 32, 8, 16256, 128, 2)):
        most, _ = api.ss_msa_plan(B, T, gamma, H, Hkv, 128, cap, api.SS_BF16)
        for _ in range(100):
            lens = [int(x) for x in rng.integers(cap // 8, cap // 2, B)]
            where, n = api.ss_msa_plan_splits(B, T, gamma, H, Hkv, 128, cap, api.SS_BF16, lens)
            assert where == 2
            args = (B, T, gamma, H, Hkv, B * most, chunk_rows, groups, lens)
            # 64 candidates between 8 and some 300 blocks lie 6 % apart, and are rounded up to whole wave groups
            assert _cut_by_hand(*args, n=n) <= 1.15 * _cut_by_hand(*args), (lens, n)


def test_cut_stands_where_little_less_than_planned_is_to_do():
    shape = lambda B, T: (B, T, 4, 32, 8, 128, 8192, api.SS_BF16)
    where = lambda B, T, lens, kept=None: api.ss_msa_plan_splits(*shape(B, T), lens, kept)[0]
    full = [8192] * 7
    assert where(8, 32, full + [8192]) == 1
    # 320 items: the whole batch's work counts
    assert where(8, 32, full + [4096]) == 1 and where(8, 32, full + [0]) == 1
    assert where(8, 32, [7168] * 8) == 1 and where(8, 32, [7136] * 8) == 2     # 7/8 of the capacity, and a block less
    assert where(8, 32, [8192] * 6 + [4096, 0]) == 2
    assert where(8, 32, full + [8192], [32] * 7 + [1]) == 1                    # one sequence pruned to one chunk of five
    assert where(8, 32, full + [8192], [26] * 8) == 1                          # fewer nodes, the same five chunks
    assert where(8, 32, full + [8192], [25] * 8) == 2                          # four chunks
    # 160 items: one sequence that is short
    assert where(4, 32, [8192] * 4) == 1 and where(4, 32, [8192] * 3 + [7000]) == 2


def test_shapes_of_the_uneven_batches_are_of_the_kind_they_stand_for():
    import test_gpu_msa_uneven as t
    for name in t.CASES:
        where, _ = api.ss_msa_plan_splits(*t._shape(name), t.CASES[name][7])
        assert where == (2 if name in t.CUT else 0), name
    plans = [api.ss_msa_plan(*t._shape(name)) for name in t.CUT]
    assert (2, 1) in plans and any(n > 2 for n, _ in plans)      # merged in the attention kernel, and by the merge kernel


def test_stages_for_the_own_rows_cost_no_resident_workgroup():
    # heads of 64 in several row chunks of nine to twelve waves: two workgroups fit a compute unit's 160 KB, whatever the tree
    # (more of the step's own rows get stages only where no workgroup goes for them)
    # (of fifteen waves the second one's ring, for it to start while the first one's last group is still at work)
    for T, gamma, H, rows, waves in ((21, 4, 40, 48, 9), (64, 2, 8, 64, 12), (64, 8, 8, 64, 12), (61, 2, 40, 80, 15), (50, 5, 8, 80, 15)):
        p = api.ss_msa_plan_launch(16, T, gamma, H, 8, 64, 4096)
        assert (p["rows_per_wave"], p["rows"], p["waves"]) == (16, rows, waves) and p["workgroups"] > 256
        assert 2 * p["lds"] <= 160 * 1024, p
    # where one workgroup fits anyway (sixteen waves: 3 rounds of own blocks; heads of 128) or the launch has one per compute
    # unit at most, the later rounds have their stages: (groups, stages and more stages per group) of 8 or 16 KB
    for shape, most_wgs, stages in (((16, 32, 4, 32, 8, 64, 4096), 1280, 2 * (3 + 2) * 8192), ((1, 21, 4, 40, 8, 64, 512), 256, 3 * (3 + 1) * 8192),
                                    ((1, 16, 4, 32, 32, 128, 2048), 256, 2 * (3 + 1) * 16384)):
        p = api.ss_msa_plan_launch(*shape)
        assert p["workgroups"] <= most_wgs and stages <= p["lds"] < stages + 4096, (shape, p)


def test_splits_of_long_trees_by_their_cost():
    # (B, T, gamma, H, Hkv) -> query rows per wave and splits of launches of 256 and more items with 32 query rows per wave
    plan = lambda B, T, gamma, H, Hkv, cap: tuple(api.ss_msa_plan_launch(B, T, gamma, H, Hkv, 128, cap)[k] for k in ("rows_per_wave", "n_splits"))
    assert plan(8, 32, 4, 32, 8, 32768) == (32, 4)      # 5 whole rounds
    assert plan(8, 32, 4, 32, 8, 8192) == (32, 4)
    assert plan(13, 27, 5, 64, 8, 4416) == (32, 1)      # short sequences: partial results cost more than a round's end
    assert plan(16, 47, 5, 40, 8, 2368) == (32, 1)
    assert plan(6, 32, 4, 40, 8, 8192) == (32, 1)
    assert plan(9, 29, 4, 32, 4, 21056)[1] > 1          # 468 items, but 5 groups of 13 on an XCD are one more than it holds
    assert plan(7, 57, 5, 28, 4, 2240) == (32, 1)       # never more than whole rounds want
    for shape in ((9, 26, 4, 48, 8, 4288), (12, 37, 6, 32, 4, 5312), (10, 24, 4, 32, 8, 5248), (8, 20, 5, 64, 8, 4096), (8, 48, 4, 32, 8, 4288),
                  (2, 59, 6, 48, 8, 9600)):
        assert plan(*shape) == (16, 1), shape           # as many rounds of 80 rows as of 96
    assert plan(12, 37, 6, 32, 4, 12288)[0] == 32       # the same rows, longer: that kernel would cut them in eight


def test_split_0_takes_no_more_than_an_equal_share():
    # it scans the step's own rows besides
    def blocks(shape):   # of split 0, of an equal share
        one = lambda u: api.ss_msa_plan_splits(*shape, api.SS_BF16, [32 * u] * shape[0])[1][0] == 1
        n, nu = api.ss_msa_plan(*shape, api.SS_BF16)[0], shape[6] // 32
        assert n > 1
        return max(u for u in range(1, nu + 1) if one(u)), -(-nu // n)
    for shape in ((1, 15, 3, 16, 16, 128, 8320), (2, 1, 5, 40, 8, 64, 9376), (1, 9, 4, 16, 16, 64, 6272), (6, 2, 3, 32, 4, 128, 2368),
                  (1, 9, 3, 32, 8, 128, 3584), (1, 4, 3, 16, 16, 128, 2912)):
        own, share = blocks(shape)
        assert own <= share, (shape, own, share)
    assert blocks((1, 16, 4, 32, 32, 128, 2048)) == (1, 8) and blocks((2, 6, 4, 32, 8, 128, 3712)) == (8, 9)   # less, where the others can take it
