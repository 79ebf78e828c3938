"""Small-tile GEMM with six and seven bands per workgroup, where it can go wrong: the accumulators beyond the sixteenth tile,
slices of k of unequal length, a last workgroup with few bands, a last row group with few rows."""
import re

import numpy as np
import pytest

import oracle
import workload as wl
from parity_util import TOL_BF16, check_forward, check_tree_kv

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SMALL = dict(n_heads=2, n_kv_heads=1, head_dim=64)


@pytest.mark.parametrize("stage,kernel,cfg,sizes", [
    # gate|up: 345 bands in sixes (the last workgroup has 3), 97 k-steps in slices of 24 and 25, 300 rows
    ("gate_up", "mid 6x3", dict(SMALL, d_model=1552, d_ffn=5520), (64,) * 4 + (44,)),
    # gate|up: 352 bands in sevens (the last has 2), 101 k-steps, 897 rows: the last group has one
    ("gate_up", "mid 7x3", dict(SMALL, d_model=1616, d_ffn=5632), (64,) * 14 + (1,)),
    # q|k|v: 400 bands in sevens (the last has 1), 101 k-steps, 300 rows
    ("qkv", "mid 7x3", dict(n_heads=120, n_kv_heads=40, head_dim=64, d_model=1616, d_ffn=64), (64,) * 4 + (44,)),
    # down: 130 bands in sixes (the last has 4), 101 k-steps, 900 rows
    ("down", "mid 6x3", dict(SMALL, d_model=4160, d_ffn=1616), (64,) * 14 + (4,)),
])
def test_tall_tiles_match_oracle(stage, kernel, cfg, sizes, monkeypatch, capfd):
    """Against the fp64 oracle with the bound of every bf16 forward: activations enter with 16 mantissa bits, K and V rows
    that round the other way are what is left."""
    from paper_2507_18181_amd.runtime import Verifier
    monkeypatch.setenv("SPECASR_DEBUG", "1")
    cfg = dict(wl.MODELS["tiny"], n_layers=1, vocab=64, **cfg)
    w = wl.make_weights(cfg, 751, "bf16")
    rng = np.random.default_rng(752)
    nb, cap, L = len(sizes), 80, 5
    K, V = wl.seeded_cache(cfg, 753, np.full(nb, L, np.int32), cap, "bf16", batch=nb)
    om = oracle.OracleModel(cfg, w)
    ver = Verifier(cfg, w, "bf16", max_nodes=64, capacity=cap, max_batch=nb)
    ver.set_cache(K, V, [L] * nb)
    trees = [wl.random_tree(rng, n, max_children=3) for n in sizes]
    toks = [rng.integers(0, cfg["vocab"], n).astype(np.int32) for n in sizes]
    capfd.readouterr()
    fw = ver.tree_forward(toks, trees)
    assert fw["status"] == 0
    plan = re.findall(r"plan %s rows=%d .*: (.+), \d+ splits" % (stage, sum(sizes)), capfd.readouterr().err)
    assert plan == [kernel]
    k1, v1 = ver.get_cache()
    for b in range(nb):
        ref = om.tree_forward(np.ascontiguousarray(K[b]), np.ascontiguousarray(V[b]), L, toks[b], trees[b])
        check_forward(ref, fw["logits"][b].cpu().numpy(), fw["argmax"][b].cpu().numpy(), TOL_BF16)
        check_tree_kv(k1[b], v1[b], L, ref, TOL_BF16)
    ver.close()
