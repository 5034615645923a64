"""Device parity against the oracle at sizes the oracle finishes in seconds.

Every device call goes through the C ABI (paper_2609_37062_amd.vsk); the
oracle is the float64 CPU statement in oracle/.
"""
import copy
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from workloads.configs import (ModelCfg, SeqSpec, Workload, decode_workload, mixed_workload,  # noqa: E402
                               prefix_groups_workload, workload)

from helpers import assert_kv_layer_local, e2e_compare  # noqa: E402

pytestmark = pytest.mark.gpu

# two layers, GQA group 4, head_dim 128: several tiles along every matrix
# and ragged row groups
MID = ModelCfg("mid-2L", n_layers=2, hidden=512, n_q_heads=8, n_kv_heads=2, head_dim=128, ffn=1536,
               vocab=2048, rope_theta=500000.0)
# hidden 2048 (64 K steps): room for up to 8 K splits of the QKV projection
WIDE = ModelCfg("wide-2L", n_layers=2, hidden=2048, n_q_heads=16, n_kv_heads=4, head_dim=128, ffn=2048,
                vocab=4096, rope_theta=500000.0)


def _run(w, **kw):
    from paper_2609_37062_amd.runner import DeviceRun
    print(f"[gpu] {w.name} seqs={w.n_seqs} rows={w.n_rows}", flush=True)
    kw.setdefault("poison_pool", True)
    d = DeviceRun(w, **kw)
    d.step()
    lg, ids = d.results()
    return d, lg, ids


def _check(w, lg, ids, subset=None, **kw):
    """End to end against the oracle: the 2e-2 bar, widened per row only where
    the oracle's own float32 run drifts further (helpers.compare_logits)."""
    st, out, kv, sub, idx, dev_rows = e2e_compare(w, lg, ids, subset, **kw)
    return st, out, kv, sub, idx


def test_config1_tiny_decode():
    w = workload(1)
    d, lg, ids = _run(w)
    st, out, kv, sub, idx = _check(w, lg, ids)
    # new K,V of every row at every layer (Invariant 1), one bf16 ulp
    assert_kv_layer_local(d, w)
    print(st)


@pytest.mark.parametrize("B", [1, 20, 70, 130])
def test_mid_decode_batches(B):
    ctx = np.random.default_rng(B).integers(0, 300, size=B)
    w = decode_workload(MID, ctx, seed=3, name=f"mid-decode-b{B}")
    d, lg, ids = _run(w)
    sub = None if B <= 20 else list(range(0, B, max(1, B // 12)))
    st, *_ = _check(w, lg, ids, sub)
    print(st)


@pytest.mark.parametrize("bps", [8, 24, 64, 512])
def test_mid_attention_splits(bps):
    """Split-K attention: one work item per KV head (bps 512) up to many
    splits merged in split order (bps 8); contexts up to 1500 tokens."""
    from paper_2609_37062_amd.runner import DeviceRun
    ctx = np.array([1499, 1, 16, 17, 700, 1023, 1024, 255])
    w = decode_workload(MID, ctx, seed=11, name=f"mid-splits-{bps}")
    print(f"[gpu] {w.name} bps={bps}", flush=True)
    d = DeviceRun(w, poison_pool=True)
    d.eng.set_tuning(0, bps)
    d.step()
    lg, ids = d.results()
    st, *_ = _check(w, lg, ids)
    print(st)


@pytest.mark.parametrize("B,shape", [(40, 0), (40, 1), (40, 2), (40, 3), (40, 4), (40, 5),
                                     (100, 0), (100, 1), (100, 2), (100, 3), (100, 4), (100, 5), (100, 6), (40, 6),
                                     (130, 0), (130, 4), (130, 5)])
def test_mid_projection_shapes(B, shape):
    """Every launch shape of the projections for 3 and 7 row groups (one or
    two 16-column tiles per wave column, a 2 x 2 wave grid, X staged in LDS
    by a loader wave) and a row-tiled pass (130 rows: 8 + 1 row groups)."""
    from paper_2609_37062_amd.runner import DeviceRun
    ctx = np.random.default_rng(100 + B).integers(0, 400, size=B)
    w = decode_workload(MID, ctx, seed=13, name=f"mid-shape-b{B}-s{shape}")
    print(f"[gpu] {w.name}", flush=True)
    d = DeviceRun(w, poison_pool=True)
    d.eng.set_tuning(3, shape)
    d.step()
    lg, ids = d.results()
    d.step()
    lg2, ids2 = d.results()
    assert np.array_equal(lg, lg2) and np.array_equal(ids, ids2)
    st, *_ = _check(w, lg, ids, list(range(0, B, max(1, B // 12))))
    print(st)


@pytest.mark.parametrize("B,target", [(9, -1), (9, 4096), (40, -1), (40, 0), (40, 4096), (100, -1), (100, 64), (100, 4096)])
def test_mid_residual_k_splits(B, target):
    """Residual projections with K split over workgroups (the splits added
    into the residual, in split order, by the RMSNorm that follows): no split
    (-1), the default (0), a few, and the most the rule allows."""
    from paper_2609_37062_amd.runner import DeviceRun
    ctx = np.random.default_rng(200 + B).integers(0, 400, size=B)
    w = decode_workload(MID, ctx, seed=17, name=f"mid-rsplit-b{B}-t{target}")
    print(f"[gpu] {w.name}", flush=True)
    d = DeviceRun(w, poison_pool=True)
    d.eng.set_tuning(5, target)
    d.step()
    lg, ids = d.results()
    d.step()
    lg2, ids2 = d.results()
    assert np.array_equal(lg, lg2) and np.array_equal(ids, ids2)
    st, *_ = _check(w, lg, ids, list(range(0, B, max(1, B // 12))))
    print(st)


# (model, rows, target) -> K splits of QKV (test_host_plans.py pins them): MID
# 40/4096 -> 2; WIDE at 3 row groups 0 (256) -> 5, 192 -> 4; at 7 row groups
# 0 (192) -> 8, 64 -> 3, 128 -> 6, 168 -> 7
@pytest.mark.parametrize("cfg,B,target", [("mid", 40, 4096), ("mid", 100, -1), ("wide", 40, -1), ("wide", 40, 0),
                                          ("wide", 40, 192), ("wide", 100, 0), ("wide", 100, 64), ("wide", 100, 128),
                                          ("wide", 100, 168)])
def test_mid_qkv_k_splits(cfg, B, target):
    """QKV with K split over workgroups (the splits' products added in split
    order by the kernel that applies rotary and writes q and the KV slots):
    no split (-1), the default (0), and 2 to 8 splits.

    MID: logits end to end, and a replay bit-exact.
    WIDE (hidden 2048, logits ~2x MID's): the checks of the full-size tests --
    each layer's new K,V within one bf16 ulp of the oracle applied to the
    device's own input residual (the values the split reduction writes), the
    residual after it, the 2e-2 bar on the head of every row, and end to end.
    End to end, one rounding flip of a query element in layer 1 moves the
    oracle's own float32 run by 0.013-0.014 on some of these rows (measured:
    10 attention outputs, then 40 MLP inputs, 482 SwiGLU products and 566
    final-norm outputs change by one ulp), so those rows take the
    float32-spread bound of compare_logits."""
    from paper_2609_37062_amd.runner import DeviceRun
    model = MID if cfg == "mid" else WIDE
    ctx = np.random.default_rng(300 + B).integers(0, 400, size=B)
    w = decode_workload(model, ctx, seed=19, name=f"{cfg}-qsplit-b{B}-t{target}")
    print(f"[gpu] {w.name}", flush=True)
    subset = list(range(0, B, max(1, B // 12)))
    if cfg == "wide":
        from test_gpu_fullsize import _check as layer_local_check
        st = layer_local_check(w, subset, tuning=[(7, target)])
        assert st["head"]["max_err"] <= 2e-2
        return
    d = DeviceRun(w, poison_pool=True)
    d.eng.set_tuning(7, target)
    d.step()
    lg, ids = d.results()
    d.step()
    lg2, ids2 = d.results()
    assert np.array_equal(lg, lg2) and np.array_equal(ids, ids2)
    st, *_ = _check(w, lg, ids, subset)
    print(st)


def test_mid_uncut_walks_past_96_blocks():
    """290 rows x 2 KV heads (580 pairs): no walk is longer than a 512th of all
    of them, so contexts of 98..107 blocks, past the 96-block split, are one
    work item each; against the oracle."""
    from paper_2609_37062_amd.runner import DeviceRun
    B = 290
    ctx = np.random.default_rng(77).integers(1560, 1700, size=B)
    w = decode_workload(MID, ctx, seed=31, name="mid-uncut")
    print(f"[gpu] {w.name}", flush=True)
    d = DeviceRun(w, poison_pool=True)
    d.step()
    assert d.eng.exec_counters()[3] == 1  # one split per row
    lg, ids = d.results()
    st, *_ = _check(w, lg, ids, [0, 17, 144, 289])
    print(st)


@pytest.mark.parametrize("lo,hi", [(900, 1000), (300, 1000)])
def test_mid_auto_split_balance(lo, hi):
    """The automatic attention split at 80 rows x 2 KV heads (160 pairs, fewer
    than the compute units): contexts within 20% of each other take one split
    per pair (no merge), a threefold spread keeps 32-block splits merged in
    split order; both against the oracle, with stale slots NaN-poisoned."""
    from paper_2609_37062_amd.runner import DeviceRun
    B = 80
    ctx = np.random.default_rng(500 + lo).integers(lo, hi, size=B)
    w = decode_workload(MID, ctx, seed=29, name=f"mid-autosplit-{lo}-{hi}")
    print(f"[gpu] {w.name}", flush=True)
    d = DeviceRun(w, poison_pool=True)
    d.step()
    lg, ids = d.results()
    d.step()
    lg2, ids2 = d.results()
    assert np.array_equal(lg, lg2) and np.array_equal(ids, ids2)
    st, *_ = _check(w, lg, ids, list(range(0, B, 7)))
    print(st)


@pytest.mark.parametrize("cfg,B,row_tile", [("mid", 130, 11), ("mid", 200, 11), ("mid", 300, 11), ("mid", 300, 8),
                                            ("mid", 300, 7), ("mid", 200, 6), ("wide", 200, 11), ("wide", 300, 7),
                                            ("wide", 130, 6)])
def test_row_tile_heights(cfg, B, row_tile):
    """Projections of a row-tiled pass at each tile height (tuning key 10;
    11 applies to gate/up and QKV, the residual projections then keep 8):
    one padded tile (130 rows: 9 groups in one tile of 11, two of 6), a
    2-group tail (200 rows at 11, 13 = 6 + 6 + 1), 11 + 8 and 7 x 2 + 5
    groups (300 rows), and the 8-group tiles at 300 rows for comparison.
    MID: logits end to end and a replay bit-exact; WIDE: the layer-local
    checks of the full-size tests (each layer's new K,V within one bf16 ulp,
    the residual, the 2e-2 head bar)."""
    from paper_2609_37062_amd.runner import DeviceRun
    model = MID if cfg == "mid" else WIDE
    ctx = np.random.default_rng(400 + B).integers(0, 400, size=B)
    w = decode_workload(model, ctx, seed=23, name=f"{cfg}-rowtile-b{B}-m{row_tile}")
    print(f"[gpu] {w.name}", flush=True)
    subset = list(range(0, B, max(1, B // 12)))
    if cfg == "wide":
        from test_gpu_fullsize import _check as layer_local_check
        st = layer_local_check(w, subset, tuning=[(10, row_tile)])
        assert st["head"]["max_err"] <= 2e-2
        return
    d = DeviceRun(w, poison_pool=True)
    d.eng.set_tuning(10, row_tile)
    d.step()
    lg, ids = d.results()
    d.step()
    lg2, ids2 = d.results()
    assert np.array_equal(lg, lg2) and np.array_equal(ids, ids2)
    st, *_ = _check(w, lg, ids, subset)
    print(st)


def test_mid_shared_prefix():
    ctx = 256 + np.random.default_rng(5).integers(3, 40, size=12)
    w = decode_workload(MID, ctx, seed=4, shared=256, name="mid-shared")
    d, lg, ids = _run(w)
    st, *_ = _check(w, lg, ids)
    print(st)


@pytest.mark.parametrize("shared,bps", [(1, 0), (0, 0), (1, 8)])
def test_mid_prefix_groups(shared, bps):
    """Two shared-prefix groups (160 and 96 tokens, one of 45 members so a
    group spans several 64-column work items, a row's query heads split
    between two of them) beside sequences of no group; prefixes read once per
    group (shared 1) or once per sequence (0)."""
    from paper_2609_37062_amd.runner import DeviceRun
    rng = np.random.default_rng(21)
    suf = rng.integers(1, 90, size=45 + 5 + 4)
    suf[3] = 0  # a member whose only private token is the new one
    w = prefix_groups_workload(MID, [(160, 45), (96, 5)], suf, seed=9, name=f"mid-groups-{shared}-{bps}")
    print(f"[gpu] {w.name}", flush=True)
    d = DeviceRun(w, poison_pool=True)
    pfx, ng = d.eng.batch_prefix_info()
    assert ng == 2 and (pfx[:45] == 10).all() and (pfx[45:50] == 6).all() and not pfx[50:].any()
    d.eng.set_tuning(4, shared)
    d.eng.set_tuning(0, bps)
    d.step()
    lg, ids = d.results()
    d.step()
    lg2, ids2 = d.results()
    assert np.array_equal(lg, lg2) and np.array_equal(ids, ids2)
    st, *_ = _check(w, lg, ids, [0, 1, 3, 20, 21, 44, 45, 47, 49, 50, 53])
    print(st)


def _graph_replays_match(d, step, n=3):
    """Capture `step` in a graph and replay it n times, with an eager pass
    between replays: every replay reproduces the eager pass bit for bit."""
    import torch
    step()
    lg1, ids1 = d.results()
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        step(stream=s.cuda_stream)
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        step(stream=torch.cuda.current_stream().cuda_stream)
    for _ in range(n):
        d.logits.zero_()
        g.replay()
        torch.cuda.synchronize()
        lg, ids = d.results()
        np.testing.assert_array_equal(lg, lg1)
        np.testing.assert_array_equal(ids, ids1)
        step()
        lg, ids = d.results()
        np.testing.assert_array_equal(lg, lg1)
    del g
    return lg1, ids1


def test_mixed_pass_graph_replay():
    """A row-tiled mixed pass (two 200-row prompts prefilled beside 6
    decodes: 406 rows, tile heights chosen by the launch rounds, prefill
    items longest first) captured in a graph: every replay, with eager
    passes between, reproduces the eager pass bit for bit, and the eager
    pass matches the oracle."""
    from paper_2609_37062_amd.runner import DeviceRun
    ctx = np.random.default_rng(71).integers(20, 300, size=6)
    w = mixed_workload(MID, n_pre=2, plen=200, ctx=ctx, seed=71, name="mid-mixed-graph")
    print(f"[gpu] {w.name}", flush=True)
    d = DeviceRun(w, poison_pool=True)
    lg, ids = _graph_replays_match(d, d.step)
    st, *_ = _check(w, lg, ids)
    print(st)
    d.release()


def test_shared_prefix_graph_replay():
    """A decode pass with shared-prefix groups captured in a graph: every
    replay, with eager passes between, reproduces the eager pass bit for bit
    (the split-merge arrival counters are back at zero after every pass)."""
    from paper_2609_37062_amd.runner import DeviceRun
    suf = np.random.default_rng(33).integers(1, 60, size=30)
    w = prefix_groups_workload(MID, [(192, 24), (64, 4)], suf, seed=33, name="mid-groups-graph")
    print(f"[gpu] {w.name}", flush=True)
    d = DeviceRun(w, poison_pool=True)
    d.eng.set_tuning(0, 8)
    d.step()
    lg1, ids1 = d.results()
    st, *_ = _check(w, lg1, ids1, [0, 5, 23, 24, 27, 28, 29])
    print(st)
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        d.step(stream=s.cuda_stream)
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        d.step(stream=torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        d.logits.zero_()
        g.replay()
        torch.cuda.synchronize()
        lg, ids = d.results()
        np.testing.assert_array_equal(lg, lg1)
        np.testing.assert_array_equal(ids, ids1)
        d.step()
        lg, ids = d.results()
        np.testing.assert_array_equal(lg, lg1)
    del g
    d.release()


@pytest.mark.parametrize("bps", [0, 8])
def test_mid_pair_boundaries(bps):
    """Decode rows whose key counts fall on and around 16-token block and
    32-key step boundaries (a wave's last step may hold one real block and a
    masked one, a block may end the sequence exactly), every unwritten pool
    slot holding a NaN pattern."""
    from paper_2609_37062_amd.runner import DeviceRun
    kv = np.array([1, 15, 16, 17, 31, 32, 33, 48, 49, 63, 64, 65, 96, 129])
    w = decode_workload(MID, kv - 1, seed=23, name=f"mid-pairs-{bps}")
    print(f"[gpu] {w.name}", flush=True)
    d = DeviceRun(w, poison_pool=True)
    d.eng.set_tuning(0, bps)
    d.step()
    lg, ids = d.results()
    st, *_ = _check(w, lg, ids)
    print(st)


def test_mid_prefix_odd_blocks():
    """Shared prefixes of an odd number of blocks (11 and 5): the two waves of
    a prefix tile split an odd number of blocks, the last step unpaired."""
    from paper_2609_37062_amd.runner import DeviceRun
    suf = np.random.default_rng(27).integers(0, 40, size=12 + 3 + 2)
    w = prefix_groups_workload(MID, [(176, 12), (80, 3)], suf, seed=27, name="mid-groups-odd")
    print(f"[gpu] {w.name}", flush=True)
    d = DeviceRun(w, poison_pool=True)
    pfx, ng = d.eng.batch_prefix_info()
    assert ng == 2 and (pfx[:12] == 11).all() and (pfx[12:15] == 5).all() and not pfx[15:].any()
    d.step()
    lg, ids = d.results()
    st, *_ = _check(w, lg, ids)
    print(st)


def test_mid_mixed_prefill_decode():
    ctx = np.random.default_rng(6).integers(10, 200, size=5)
    w = mixed_workload(MID, n_pre=2, plen=45, ctx=ctx, seed=7, name="mid-mixed")
    d, lg, ids = _run(w)
    st, out, kv, sub, idx = _check(w, lg, ids)
    # every prefill row wrote its own K,V at every layer, one bf16 ulp
    assert_kv_layer_local(d, w)
    print(st)


@pytest.mark.parametrize("prefill_kernel", [1, 0])
def test_mid_chunked_prefill_with_context(prefill_kernel):
    """Prefill chunks that continue cached sequences (rows at positions
    ctx..ctx+q-1 attend the cache and the chunk's own earlier rows), a fresh
    prompt, a two-row chunk and decode rows in one pass; the causal
    multi-row kernel (1) and one work item per row (0)."""
    from paper_2609_37062_amd.runner import DeviceRun
    rng = np.random.default_rng(31)
    specs = [(100, 37), (0, 50), (300, 1), (17, 2), (33, 1), (250, 45)]
    n_pool = 120
    perm = [int(b) for b in rng.permutation(n_pool)]
    seqs, pos = [], 0
    for i, (ctx, q) in enumerate(specs):
        nb = (ctx + 15) // 16
        seqs.append(SeqSpec(ctx, q, perm[pos:pos + nb], [(0, ctx, i)] if ctx else []))
        pos += nb
    tokens = rng.integers(0, MID.vocab, size=sum(q for _, q in specs)).astype(np.int32)
    w = Workload(0, f"mid-chunked-{prefill_kernel}", MID, seqs, n_pool, tokens, 5)
    print(f"[gpu] {w.name}", flush=True)
    d = DeviceRun(w, poison_pool=True)
    d.eng.set_tuning(6, prefill_kernel)
    d.step()
    lg, ids = d.results()
    d.step()
    lg2, ids2 = d.results()
    assert np.array_equal(lg, lg2) and np.array_equal(ids, ids2)
    st, out, kv, sub, idx = _check(w, lg, ids)
    assert_kv_layer_local(d, w)
    print(st)


@pytest.mark.parametrize("kind", ["decode", "chunk"])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("own", [30, 700])
def test_shared_blocks_equal_copies(kind, head_dim, own):
    """Rows behind one common prefix that is not folded (key 4 at 0, or decode
    rows beside a prompt) read its blocks many times, with ordinary loads where
    they are at least half of all blocks (30 own tokens) and non-temporal ones
    where they are less (700): bit for bit the same pass as with a copy of the
    prefix per sequence, where no block is read twice."""
    from paper_2609_37062_amd.runner import DeviceRun
    model = dataclasses.replace(MID, name=f"mid-hd{head_dim}", head_dim=head_dim)
    prefix, n = 320, 6
    rng = np.random.default_rng(own + head_dim)
    ctx = [prefix + own + int(x) for x in rng.integers(0, 20, size=n)]
    got = []
    for shared in (True, False):
        perm = [int(b) for b in np.random.default_rng(3).permutation(600)]
        take = lambda tokens: [perm.pop() for _ in range((tokens + 15) // 16)]  # noqa: E731
        seqs = [SeqSpec(0, 21, [], [])] if kind == "chunk" else []
        common = take(prefix)
        for i, c in enumerate(ctx):
            seqs.append(SeqSpec(c, 1, (common if shared else take(prefix)) + take(c + 1 - prefix),
                                [(0, prefix, 1000), (prefix, c - prefix, i)]))
        tokens = np.random.default_rng(4).integers(0, model.vocab, size=sum(q.q_len for q in seqs)).astype(np.int32)
        w = Workload(0, f"copies-{kind}-{head_dim}-{own}-{shared}", model, seqs, 600, tokens, 6)
        print(f"[gpu] {w.name}", flush=True)
        d = DeviceRun(w, poison_pool=True)
        d.eng.set_tuning(4, 0)
        d.step()
        got.append(d.results())
        if shared:
            _check(w, *got[0])
        d.release()
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])


def test_replay_is_idempotent_and_deterministic():
    ctx = np.random.default_rng(8).integers(20, 400, size=24)
    w = decode_workload(MID, ctx, seed=9)
    d, lg1, ids1 = _run(w)
    K1, V1 = d.read_kv(1, d.eng.batch_host()["slot"])
    for _ in range(3):
        d.step()
    lg2, ids2 = d.results()
    K2, V2 = d.read_kv(1, d.eng.batch_host()["slot"])
    np.testing.assert_array_equal(lg1, lg2)
    np.testing.assert_array_equal(ids1, ids2)
    np.testing.assert_array_equal(K1, K2)
    np.testing.assert_array_equal(V1, V2)


def test_block_permutation_is_bitwise_invariant():
    ctx = np.random.default_rng(10).integers(20, 300, size=9)
    w = decode_workload(MID, ctx, seed=11)
    _, lg1, ids1 = _run(w)
    w2 = copy.deepcopy(w)
    perm = np.random.default_rng(12).permutation(w.n_pool_blocks)
    for s in w2.seqs:
        s.blocks = [int(perm[b]) for b in s.blocks]
    _, lg2, ids2 = _run(w2)
    np.testing.assert_array_equal(lg1, lg2)
    np.testing.assert_array_equal(ids1, ids2)


def test_batch_row_order_is_bitwise_invariant():
    ctx = np.random.default_rng(13).integers(20, 300, size=10)
    w = decode_workload(MID, ctx, seed=14)
    _, lg1, ids1 = _run(w)
    order = np.random.default_rng(15).permutation(10)
    w2 = copy.deepcopy(w)
    w2.seqs = [w.seqs[i] for i in order]
    for j, i in enumerate(order):
        w2.seqs[j].content = [(p0, n, int(i)) for (p0, n, _c) in w.seqs[i].content]
    w2.tokens = w.tokens[order]
    _, lg2, ids2 = _run(w2)
    np.testing.assert_array_equal(lg1[order], lg2)
    np.testing.assert_array_equal(ids1[order], ids2)
