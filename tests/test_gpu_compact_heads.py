"""In-place compaction with several heads per block: head groups that are not full, groups that take more than one turn, and
rows too large to stage at once."""
import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype,kv_heads,head_dim,length", [
    ("bf16", 3, 64, 2), ("bf16", 10, 128, 9), ("bf16", 8, 128, 40), ("f32", 9, 64, 64), ("f32", 2, 256, 40),
])
def test_accepted_rows_move_to_the_front(dtype, kv_heads, head_dim, length):
    """Against a gather on the host; every row outside the moves keeps its bits."""
    from paper_2507_18181_amd.runtime import Verifier
    cfg = dict(wl.MODELS["tiny"], n_layers=2, d_model=16, d_ffn=16, n_heads=kv_heads, n_kv_heads=kv_heads, head_dim=head_dim, vocab=8)
    ver = Verifier(cfg, wl.make_weights(cfg, 751, dtype), dtype, max_nodes=64, capacity=90, max_batch=2)
    rng = np.random.default_rng(752)
    K, V = wl.seeded_cache(cfg, 753, np.full(2, 90, np.int32), 90, dtype, batch=2)
    Ls = [4, 25]
    ver.set_cache(K, V, Ls)
    # one sequence whose rows all stay, one whose path leaves the front and overlaps its sources
    rest = np.sort(rng.choice(np.arange(1, 64), length - 1, replace=False))
    paths = [list(range(length)), [0] + rest.tolist()]
    assert ver.commit([64, 64], paths) == 0
    k1, v1 = ver.get_cache()
    for b, (L, p) in enumerate(zip(Ls, paths)):
        for before, after in ((K, k1), (V, v1)):
            want = before[b].copy()
            want[:, :, L:L + length] = before[b][:, :, L + np.asarray(p)]
            assert np.array_equal(after[b], want)
        assert ver.kv_len[b] == L + length
    ver.close()
