"""One layer of each model class that is measured, at the row counts where the GEMM planners change kernels: every kernel
instance that such a model runs is compared with the oracle, and the plan itself is pinned, so that another
constant in a planner cannot move a test off its kernel."""
import re

import numpy as np
import pytest

import oracle
import workload as wl
from parity_util import TOL_BF16, check_forward, check_tree_kv

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# rows: kernel and splits of q|k|v, o, gate|up, down (slice: half-bands x 16 rows, 0: 8 rows with both
# activation planes in one operand; mid: bands x 32 rows, pair: bands x 32 rows, skinny: ring)
PLANS = {
    ("1b", 1): "slice 1x0 1, slice 1x0 1, slice 3x0 1, slice 2x0 4",
    ("1b", 8): "slice 1x0 1, slice 1x0 1, slice 3x0 1, slice 2x0 4",
    ("1b", 16): "slice 1x1 1, slice 1x1 1, slice 3x1 1, slice 2x1 4",
    ("1b", 24): "slice 1x2 1, slice 1x2 1, slice 3x2 1, skinny 4 16",
    ("1b", 37): "skinny 8 2, skinny 4 4, slice 3x3 1, slice 4x3 8",
    ("1b", 64): "skinny 8 2, skinny 4 4, skinny 8 2, slice 4x4 8",
    ("1b", 72): "mid 2x2 3, mid 2x2 4, mid 2x3 1, mid 2x3 8",
    ("1b", 160): "mid 3x3 4, mid 2x3 4, mid 3x3 1, mid 3x3 5",
    ("1b", 384): "mid 3x3 2, mid 2x3 2, mid 6x3 1, wide 8",
    ("1b", 1024): "wide 3, mid 3x3 1, wide 2, wide 4",
    ("7b", 1): "slice 3x0 1, slice 1x0 1, slice 6x0 1, slice 2x0 2",
    ("7b", 5): "slice 3x0 1, slice 1x0 1, slice 6x0 1, slice 2x0 2",
    ("7b", 8): "slice 3x0 1, slice 1x0 1, slice 6x0 1, slice 2x0 2",
    ("7b", 32): "slice 3x2 1, slice 1x2 1, slice 6x2 1, skinny 12 8",
    ("7b", 40): "skinny 8 4, skinny 8 4, slice 6x3 1, slice 4x3 4",
    ("7b", 64): "skinny 8 4, skinny 8 4, mid 3x2 1, mid 3x2 5",
    ("7b", 87): "mid 3x3 2, mid 3x3 5, mid 3x3 1, mid 3x3 5",
    ("7b", 128): "wide 5, mid 2x2 2, wide 2, wide 13",
    ("7b", 384): "mid 6x3 1, wide 5, pair 10x4 1, wide 5",
    ("7b", 810): "mid 7x3 1, wide 2, pair 10x4 1, wide 2",
    ("13b", 2): "slice 4x0 1, skinny 8 8, slice 7x0 1, slice 4x0 3",
    ("13b", 8): "slice 4x0 1, skinny 8 8, slice 7x0 1, slice 4x0 3",
    ("13b", 9): "slice 4x1 1, skinny 8 8, slice 7x1 1, slice 4x1 3",
    ("13b", 32): "slice 4x2 1, skinny 8 8, slice 7x2 1, skinny 8 16",
    ("13b", 48): "skinny 8 8, mid 3x2 4, skinny 8 8, skinny 8 16",
    ("13b", 80): "wide 4, mid 3x3 4, wide 2, wide 12",
}


@pytest.mark.parametrize("model,sizes", [
    ("1b", (1,)), ("1b", (8,)), ("1b", (16,)), ("1b", (24,)), ("1b", (37,)), ("1b", (64,)), ("1b", (40, 32)), ("1b", (64, 64, 32)), ("1b", (64,) * 6), ("1b", (64,) * 16),
    ("7b", (1,)), ("7b", (5,)), ("7b", (8,)), ("7b", (32,)), ("7b", (40,)), ("7b", (64,)), ("7b", (24, 21, 23, 19)), ("7b", (64, 64)), ("7b", (64,) * 6), ("7b", (64,) * 12 + (42,)),
    ("13b", (2,)), ("13b", (8,)), ("13b", (9,)), ("13b", (32,)), ("13b", (48,)), ("13b", (40, 40)),
])
def test_one_layer_against_the_oracle(model, sizes, monkeypatch, capfd):
    from paper_2507_18181_amd.runtime import Verifier
    monkeypatch.setenv("SPECASR_DEBUG", "1")
    cfg = dict(wl.MODELS[model], n_layers=1, vocab=64)
    w = wl.make_weights(cfg, 811, "bf16")
    rng = np.random.default_rng([812, sum(sizes)])
    nb, cap = len(sizes), 128
    Ls = [int(x) for x in rng.integers(0, 40, nb)]
    K, V = wl.seeded_cache(cfg, 813, np.asarray(Ls, np.int32), cap, "bf16", batch=nb)
    om = oracle.OracleModel(cfg, w)
    ver = Verifier(cfg, w, "bf16", max_nodes=64, capacity=cap, max_batch=nb)
    ver.set_cache(K, V, Ls)
    trees = [wl.random_tree(rng, n, max_children=3) for n in sizes]
    toks = [rng.integers(0, cfg["vocab"], n).astype(np.int32) for n in sizes]
    capfd.readouterr()
    fw = ver.tree_forward(toks, trees)
    assert fw["status"] == 0
    plan = re.findall(r"plan (\w+) rows=%d .*: (.+), (\d+) splits" % sum(sizes), capfd.readouterr().err)
    got = ", ".join("%s %s" % (k, s) for n, k, s in plan if n != "lm_head")
    print("plan", (model, sum(sizes)), repr(got))
    k1, v1 = ver.get_cache()
    for b in range(nb):
        ref = om.tree_forward(np.ascontiguousarray(K[b]), np.ascontiguousarray(V[b]), Ls[b], toks[b], trees[b])
        check_forward(ref, fw["logits"][b].cpu().numpy(), fw["argmax"][b].cpu().numpy(), TOL_BF16)
        check_tree_kv(k1[b], v1[b], Ls[b], ref, TOL_BF16)
    ver.close()
    assert got == PLANS[model, sum(sizes)]
