"""Calls with 33 to a few hundred tree nodes: the small-tile GEMM and the unsplit tiled gate|up at the edges of
their tiles (groups of 32 rows, 2 .. 3 groups and bands per workgroup, k slices shorter than the ring)."""
import numpy as np
import pytest

import oracle
import workload as wl
from parity_util import TOL_BF16, check_forward, check_tree_kv

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape", [
    dict(d_model=1040, d_ffn=2064, n_heads=16, n_kv_heads=4, head_dim=64),   # 65 / 129 k-steps, 129 gate|up bands
    dict(d_model=544, d_ffn=4496, n_heads=5, n_kv_heads=5, head_dim=128),    # 34 / 281 k-steps, 281 bands
    dict(d_model=512, d_ffn=528, n_heads=6, n_kv_heads=3, head_dim=64),      # 32 / 33 k-steps: one k-split only
])
def test_row_counts_around_the_tiles(shape):
    """Every sequence against the fp64 oracle run on it alone; the bound is the regression guard of
    check_forward (activations enter with 16 mantissa bits)."""
    from paper_2507_18181_amd.runtime import Verifier
    cfg = dict(wl.MODELS["tiny"], n_layers=1, vocab=65, **shape)
    w = wl.make_weights(cfg, 611, "bf16")
    rng = np.random.default_rng(612)
    om = oracle.OracleModel(cfg, w)
    nb, cap = 4, 128
    Ls = [40, 0, 21, 33]
    K, V = wl.seeded_cache(cfg, 613, np.asarray(Ls, np.int32), cap, "bf16", batch=nb)
    ver = Verifier(cfg, w, "bf16", max_nodes=64, capacity=cap, max_batch=nb)
    for sizes in ((30, 1, 1, 1), (45, 1, 1, 1), (50, 10, 2, 2), (60, 3, 1, 1), (64, 16, 8, 8), (64, 20, 12, 1), (64, 32, 20, 12), (33, 64, 31, 1), (64, 64, 64, 1), (64, 64, 64, 64)):
        trees = [wl.random_tree(rng, n, max_children=3) for n in sizes]
        toks = [rng.integers(0, cfg["vocab"], n).astype(np.int32) for n in sizes]
        ver.set_cache(K, V, Ls)
        fw = ver.tree_forward(toks, trees)
        assert fw["status"] == 0
        k1, v1 = ver.get_cache()
        for b in range(nb):
            ref = om.tree_forward(np.ascontiguousarray(K[b]), np.ascontiguousarray(V[b]), Ls[b], toks[b], trees[b])
            check_forward(ref, fw["logits"][b].cpu().numpy(), fw["argmax"][b].cpu().numpy(), TOL_BF16)
            check_tree_kv(k1[b], v1[b], Ls[b], ref, TOL_BF16)
    ver.close()
