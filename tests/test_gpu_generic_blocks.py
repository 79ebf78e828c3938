"""The linears of the dtype-generic path that read their input from memory: 4 blocks of 256 inputs asked for at once up to 512
workgroups, 2 above; inputs that end inside, at and behind a round of blocks."""
import numpy as np
import pytest

import oracle
import workload as wl
from parity_util import check_tree_kv, row_rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d_model,d_ffn,sizes", [
    (520, 2056, (1, 56, 64)),   # down: 65 x 1, 65 x 7 = 455 and 65 x 8 = 520 workgroups; 8 blocks and a remainder of 8 inputs
    (72, 1024, (8,)),           # one whole round of 4
    (72, 1032, (9,)),           # and 8 inputs of the next
    (72, 776, (16,)),           # 3 blocks and 8 inputs
])
def test_rounds_of_blocks(d_model, d_ffn, sizes):
    """fp32 against the fp64 oracle: sums of at most 2056 terms, 2^-24 * sqrt(2056) = 2.7e-6 each."""
    from paper_2507_18181_amd.runtime import Verifier
    cfg = dict(wl.MODELS["tiny"], n_layers=1, d_model=d_model, d_ffn=d_ffn, n_heads=4, n_kv_heads=2, head_dim=32, vocab=65)
    w = wl.make_weights(cfg, 721, "f32")
    rng = np.random.default_rng([722, d_ffn])
    L, cap = 20, 96
    om = oracle.OracleModel(cfg, w)
    ver = Verifier(cfg, w, "f32", max_nodes=64, capacity=cap)
    K, V = wl.seeded_cache(cfg, 723, L, cap, "f32")
    for n in sizes:
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
