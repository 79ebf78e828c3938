"""The dtype-generic linears on both sides of the width up to which a workgroup normalises its input rows itself."""
import numpy as np
import pytest

import oracle
import workload as wl
from parity_util import check_tree_kv, row_rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("d_model", [8, 256, 264, 1024, 1032])
def test_linears_that_normalise_their_input(d_model):
    """fp32 against the fp64 oracle, with 8 rows per workgroup full, part-filled and single, and rotary pairs and
    key/value heads that end inside a workgroup.  Sums of at most 1032 terms: a few 2^-24 * sqrt(1032) per layer."""
    from paper_2507_18181_amd.runtime import Verifier
    cfg = dict(wl.MODELS["tiny"], n_layers=2, d_model=d_model, d_ffn=24, n_heads=3, n_kv_heads=1, head_dim=8, vocab=9)
    w = wl.make_weights(cfg, 721, "f32")
    rng = np.random.default_rng(722)
    L, cap = 11, 40
    om = oracle.OracleModel(cfg, w)
    ver = Verifier(cfg, w, "f32", max_nodes=64, capacity=cap)
    K, V = wl.seeded_cache(cfg, 723, L, cap, "f32")
    for n in (1, 7, 8, 9, 17):
        parents = wl.random_tree(rng, n, max_children=3)
        tokens = rng.integers(0, cfg["vocab"], n).astype(np.int32)
        ver.set_cache(K, V, [L])
        ref = om.tree_forward(np.ascontiguousarray(K[0]), np.ascontiguousarray(V[0]), L, tokens, parents)
        fw = ver.tree_forward([tokens], [parents])
        assert fw["status"] == 0
        assert row_rel_err(fw["logits"][0].cpu().numpy()[:n], ref["logits"]).max() <= 1e-5
        # the same without logits in the caller's array, and the draft-side read-out with them
        assert torch.equal(ver.tree_forward([tokens], [parents], want_logits=False)["argmax"], fw["argmax"])
        top = ver.tree_forward_top2([tokens], [parents], want_logits=True)
        assert torch.equal(top["logits"][0, :n], fw["logits"][0, :n])
        assert torch.equal(top["top2"][0, :n, 0], fw["argmax"][0, :n])
        k1, v1 = ver.get_cache()
        check_tree_kv(k1[0], v1[0], L, ref, 1e-5)
    ver.close()


@pytest.mark.parametrize("d_model,sizes", [(16, (64,) * 4), (16, (64,) * 4 + (1,)), (520, (64,) * 4 + (4,)), (520, (64,) * 4 + (5,))])
def test_many_rows_on_both_sides_of_the_line(d_model, sizes):
    """fp32 against the fp64 oracle at the number of rows from which the norm is a kernel of its own."""
    from paper_2507_18181_amd.runtime import Verifier
    cfg = dict(wl.MODELS["tiny"], n_layers=2, d_model=d_model, d_ffn=24, n_heads=3, n_kv_heads=1, head_dim=8, vocab=9)
    w = wl.make_weights(cfg, 725, "f32")
    rng = np.random.default_rng(726)
    L, cap, nb = 11, 80, len(sizes)
    om = oracle.OracleModel(cfg, w)
    ver = Verifier(cfg, w, "f32", max_nodes=64, capacity=cap, max_batch=nb)
    K, V = wl.seeded_cache(cfg, 727, np.full(nb, L, np.int32), cap, "f32", batch=nb)
    ver.set_cache(K, V, [L] * nb)
    trees = [wl.random_tree(rng, n, max_children=3) for n in sizes]
    toks = [rng.integers(0, cfg["vocab"], n).astype(np.int32) for n in sizes]
    fw = ver.tree_forward(toks, trees)
    assert fw["status"] == 0
    k1, v1 = ver.get_cache()
    for b, n in enumerate(sizes):
        ref = om.tree_forward(np.ascontiguousarray(K[b]), np.ascontiguousarray(V[b]), L, toks[b], trees[b])
        assert row_rel_err(fw["logits"][b].cpu().numpy()[:n], ref["logits"]).max() <= 1e-5
        check_tree_kv(k1[b], v1[b], L, ref, 1e-5)
    ver.close()
