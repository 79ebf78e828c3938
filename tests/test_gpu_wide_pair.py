"""gate|up of wide passes with k halved inside the workgroup, where it can go wrong: one k-step, an odd number of them, fewer
than the ring holds, bands and rows that do not fill the last tile."""
import re

import numpy as np
import pytest

import oracle
import workload as wl
from parity_util import TOL_BF16, check_forward, check_tree_kv

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kernel,d_model,d_ffn,sizes", [
    ("pair 10x4", 16, 6912, (64,) * 8 + (3,)),    # 1 k-step: the second half has none; 432 bands, 515 rows
    ("pair 10x4", 96, 6912, (64,) * 8 + (3,)),    # 3 steps per half, as many as ring stages
    ("pair 10x4", 112, 6928, (64,) * 10),         # 4 and 3 steps; 433 bands
    ("pair 8x4", 272, 1072, (64, 64, 1)),         # 9 and 8 steps, ring of 4; 67 bands, 129 rows
    ("pair 8x4", 320, 1072, (64,) * 6 + (36,)),   # 10 steps, two more than two turns of the ring; 420 rows
])
def test_halved_k_matches_oracle(kernel, d_model, d_ffn, sizes, monkeypatch, capfd):
    """Against the fp64 oracle with the bound of every bf16 forward: activations enter with 16 mantissa bits, K and V rows
    that round the other way are what is left."""
    from paper_2507_18181_amd.runtime import Verifier
    monkeypatch.setenv("SPECASR_DEBUG", "1")
    cfg = dict(wl.MODELS["tiny"], n_layers=1, d_model=d_model, d_ffn=d_ffn, n_heads=1, n_kv_heads=1, head_dim=64, vocab=64)
    w = wl.make_weights(cfg, 741, "bf16")
    rng = np.random.default_rng(742)
    nb, cap, L = len(sizes), 80, 5
    K, V = wl.seeded_cache(cfg, 743, np.full(nb, L, np.int32), cap, "bf16", batch=nb)
    om = oracle.OracleModel(cfg, w)
    ver = Verifier(cfg, w, "bf16", max_nodes=64, capacity=cap, max_batch=nb)
    ver.set_cache(K, V, [L] * nb)
    trees = [wl.random_tree(rng, n, max_children=3) for n in sizes]
    toks = [rng.integers(0, cfg["vocab"], n).astype(np.int32) for n in sizes]
    capfd.readouterr()
    fw = ver.tree_forward(toks, trees)
    assert fw["status"] == 0
    assert re.findall(r"plan gate_up rows=%d .*: (.+), \d+ splits" % sum(sizes), capfd.readouterr().err) == [kernel]
    k1, v1 = ver.get_cache()
    for b in range(nb):
        ref = om.tree_forward(np.ascontiguousarray(K[b]), np.ascontiguousarray(V[b]), L, toks[b], trees[b])
        check_forward(ref, fw["logits"][b].cpu().numpy(), fw["argmax"][b].cpu().numpy(), TOL_BF16)
        check_tree_kv(k1[b], v1[b], L, ref, TOL_BF16)
    ver.close()
