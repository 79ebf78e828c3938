"""The tree attention at the edges of its tiling: tiles that the prefix, the tree and the end of the
keys cut in every position, wavefronts with none, one and several tiles, one chunk and several, and
sequences of a batch in another order than their length."""
import numpy as np
import pytest

import oracle
import workload as wl
from parity_util import TOL_BF16, check_forward, check_tree_kv

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("head_dim", [64, 128])
def test_single_sequence_key_counts(head_dim):
    """Against the fp64 oracle; the bound is the regression guard of check_forward (queries and
    probabilities enter with 16 mantissa bits).  704 keys is where one chunk ends, 1280 where the
    smallest chunk grows."""
    from paper_2507_18181_amd.runtime import Verifier
    cfg = dict(wl.MODELS["tiny"], n_layers=1, d_model=128, n_heads=4, n_kv_heads=2, head_dim=head_dim, d_ffn=96, vocab=61)
    w = wl.make_weights(cfg, 411, "bf16")
    # larger query and key weights: scores of several units, so that the running maximum moves
    for k in ("wq", "wk"):
        w["layers"][0][k] = wl.bf16_bits(wl.bf16_to_f32(w["layers"][0][k]) * 6)
    rng = np.random.default_rng(412)
    cap = 1400
    om = oracle.OracleModel(cfg, w)
    ver = Verifier(cfg, w, "bf16", max_nodes=64, capacity=cap)
    K, V = wl.seeded_cache(cfg, 413, cap - 64, cap, "bf16")
    for L, n in ((0, 1), (0, 64), (31, 1), (32, 33), (33, 31), (97, 64), (128, 5), (160, 17), (640, 64), (641, 64), (700, 9), (1279, 2), (1330, 64)):
        parents = wl.random_tree(rng, n, max_children=3)
        tokens = rng.integers(0, cfg["vocab"], n).astype(np.int32)
        ver.set_cache(K, V, [L])
        ref = om.tree_forward(np.ascontiguousarray(K[0]), np.ascontiguousarray(V[0]), L, tokens, parents)
        fw = ver.tree_forward([tokens], [parents])
        assert fw["status"] == 0
        check_forward(ref, fw["logits"][0].cpu().numpy(), fw["argmax"][0].cpu().numpy(), TOL_BF16)
        k1, v1 = ver.get_cache()
        check_tree_kv(k1[0], v1[0], L, ref, TOL_BF16)
    ver.close()


@pytest.mark.parametrize("head_dim,kv_heads,batch", [(64, 1, 17), (128, 4, 16), (64, 2, 3)])
def test_batches_of_unsorted_lengths(head_dim, kv_heads, batch):
    """Up to 16 sequences travel in the kernel arguments sorted by length, more are read from memory;
    with few (KV head, sequence, row group) triples the keys are chunked, with many they are not."""
    from paper_2507_18181_amd.runtime import Verifier
    cfg = dict(wl.MODELS["tiny"], n_layers=1, d_model=128, n_heads=2 * kv_heads, n_kv_heads=kv_heads, head_dim=head_dim, d_ffn=96, vocab=61)
    w = wl.make_weights(cfg, 421, "bf16")
    rng = np.random.default_rng([422, batch])
    Ls = [int(x) for x in rng.integers(0, 500, batch)]
    Ls[0], Ls[-1] = 3, 511
    sizes = [int(x) for x in rng.integers(1, 41, batch)]
    sizes[0] = 64
    cap = 600
    om = oracle.OracleModel(cfg, w)
    ver = Verifier(cfg, w, "bf16", max_nodes=64, capacity=cap, max_batch=batch)
    K, V = wl.seeded_cache(cfg, 423, np.asarray(Ls, np.int32), cap, "bf16", batch=batch)
    ver.set_cache(K, V, Ls)
    trees = [wl.random_tree(rng, n, max_children=3) for n in sizes]
    toks = [rng.integers(0, cfg["vocab"], n).astype(np.int32) for n in sizes]
    fw = ver.tree_forward(toks, trees)
    assert fw["status"] == 0
    for b in range(batch):
        ref = om.tree_forward(np.ascontiguousarray(K[b]), np.ascontiguousarray(V[b]), Ls[b], toks[b], trees[b])
        check_forward(ref, fw["logits"][b].cpu().numpy(), fw["argmax"][b].cpu().numpy(), TOL_BF16)
    ver.close()
