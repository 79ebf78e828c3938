"""The dtype-generic kernels where their shared launches and unrolled loops end: output counts that are
no multiple of a block, q, k and v of different sizes, key counts around the 256-key chunk and 8-row step."""
import numpy as np
import pytest

import oracle
import workload as wl
from parity_util import check_tree_kv, row_rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape", [
    dict(d_model=24, d_ffn=40, n_heads=3, n_kv_heads=1, head_dim=8, vocab=7),
    dict(d_model=264, d_ffn=520, n_heads=2, n_kv_heads=1, head_dim=256, vocab=1),
    dict(d_model=72, d_ffn=8, n_heads=5, n_kv_heads=5, head_dim=16, vocab=33),
])
def test_generic_kernels_match_oracle(shape):
    """fp32 against the fp64 oracle: sums of at most 520 terms, so a few 2^-24 * sqrt(520) per layer."""
    from paper_2507_18181_amd.runtime import Verifier
    cfg = dict(wl.MODELS["tiny"], n_layers=2, **shape)
    w = wl.make_weights(cfg, 711, "f32")
    rng = np.random.default_rng(712)
    cap = 330
    om = oracle.OracleModel(cfg, w)
    ver = Verifier(cfg, w, "f32", max_nodes=64, capacity=cap)
    K, V = wl.seeded_cache(cfg, 713, cap - 64, cap, "f32")
    for L, n in ((0, 1), (3, 8), (6, 9), (240, 16), (248, 17), (255, 2), (266, 64)):
        parents = wl.random_tree(rng, n, max_children=3)
        tokens = rng.integers(0, cfg["vocab"], n).astype(np.int32)
        ver.set_cache(K, V, [L])
        ref = om.tree_forward(np.ascontiguousarray(K[0]), np.ascontiguousarray(V[0]), L, tokens, parents)
        fw = ver.tree_forward([tokens], [parents])
        assert fw["status"] == 0
        assert row_rel_err(fw["logits"][0].cpu().numpy()[:n], ref["logits"]).max() <= 1e-5
        k1, v1 = ver.get_cache()
        check_tree_kv(k1[0], v1[0], L, ref, 1e-5)
    ver.close()
