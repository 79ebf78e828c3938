"""Acceptance that merges the argmax records of a vocabulary's parts, with one thread per node and with 16: 16, 17 and many
records, ties between them, every node of the tree."""
import numpy as np
import pytest

import oracle
import workload as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("vocab", [16384, 16385, 17409, 32767, 152064])
def test_verify_takes_the_lowest_of_the_largest_ids(vocab):
    """Records of 1024 ids.  lm_head has 60 different rows, the later ones in fewer and fewer places, so the largest logit of a
    node stands in many parts or in few; the returned logits say where."""
    from paper_2507_18181_amd.runtime import Verifier
    cfg = dict(wl.MODELS["tiny"], n_layers=1, d_model=64, n_heads=1, n_kv_heads=1, head_dim=64, d_ffn=64, vocab=vocab)
    w = wl.make_weights(cfg, 521, "bf16")
    rng = np.random.default_rng([522, vocab])
    kind = np.minimum(rng.geometric(0.12, vocab) - 1, 59)
    w["lm_head"] = np.ascontiguousarray(np.asarray(w["lm_head"])[:60][kind])
    sizes = (64, 1, 23)
    ver = Verifier(cfg, w, "bf16", max_nodes=64, capacity=80, max_batch=3)
    trees = [wl.random_tree(rng, n, max_children=3) for n in sizes]
    toks = [rng.integers(0, vocab, n).astype(np.int32) for n in sizes]
    for turn in range(2):
        ver.kv_len[:] = 0
        out = ver.verify_tree(toks, trees, want_logits=True)
        assert out["status"] == 0
        lg = out["logits"].cpu().numpy()
        parts = set()
        for b, n in enumerate(sizes):
            want = lg[b, :n].argmax(1)   # the first of the largest
            parts |= set((want // 1024).tolist())
            assert np.array_equal(out["argmax"][b, :n], want)
            path, alen, nxt = oracle.accept(toks[b], trees[b], want.astype(np.int32))
            assert (out["accept_len"][b], out["next_token"][b]) == (alen, nxt)
            assert out["path"][b, :alen].tolist() == path.tolist() and (out["path"][b, alen:] == -1).all()
            for i in range(1, n):   # the second turn follows the target: some drafts are accepted
                if i % 4:
                    toks[b][i] = want[trees[b][i]]
        assert len(parts) > 1
    assert out["accept_len"].max() > 1
    ver.close()


@pytest.mark.parametrize("vocab", [65536, 65537, 131075])
def test_accept_from_logits_with_many_pieces(vocab):
    """Records of 4096 ids: 16, 17 and 33 of them; ties between them, infinities and NaN."""
    from paper_2507_18181_amd.runtime import Verifier
    cfg = dict(wl.MODELS["tiny"], n_layers=1, d_model=8, n_heads=1, n_kv_heads=1, head_dim=8, d_ffn=8, vocab=vocab)
    ver = Verifier(cfg, wl.make_weights(cfg, 523, "f32"), "f32", max_nodes=64, capacity=64, max_batch=2)
    rng = np.random.default_rng([524, vocab])
    sizes = (64, 37)
    trees = [wl.random_tree(rng, n, max_children=3) for n in sizes]
    toks = [rng.integers(0, vocab, n).astype(np.int32) for n in sizes]
    lg = rng.integers(-3, 4, (2, 64, vocab)).astype(np.float32)
    lg[0, 1] = -np.inf
    lg[0, 2] = np.nan
    lg[0, 3] = -np.inf
    lg[0, 3, vocab - 1] = -1e30
    for i in range(8, 64):
        lg[:, i, rng.integers(0, vocab, 3)] = 9.0   # a tie of three ids anywhere
    lg[1, 5, 4096::4096] = np.inf
    want = np.where(np.isnan(lg), -np.inf, lg).argmax(2).astype(np.int32)
    for b, n in enumerate(sizes):
        for i in range(1, n):
            if i % 3:
                toks[b][i] = want[b, trees[b][i]]
    out = ver.accept(toks, trees, logits_dev=torch.from_numpy(lg).to(ver.device))
    assert out["status"] == 0
    am = out["argmax"].cpu().numpy()
    for b, n in enumerate(sizes):
        assert np.array_equal(am[b, :n], want[b, :n])
        path, alen, nxt = oracle.accept(toks[b], trees[b], want[b, :n])
        assert (out["accept_len"][b], out["next_token"][b]) == (alen, nxt)
        assert out["path"][b, :alen].tolist() == path.tolist()
    ver.close()
