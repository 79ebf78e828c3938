"""The bits of a forward.  Every sum of these kernels has one order and every product that meets a sum is fused or not by what the source
says, so a change that only schedules, merges or moves work leaves logits and cache rows as they are.  Digests of both, per kernel path;
a change that means to reorder a sum replaces the digests of the paths it touches and says so."""
import hashlib

import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CLASS = dict(n_layers=2, d_model=2048, n_heads=32, n_kv_heads=4, head_dim=64, d_ffn=5632, vocab=1000, rms_eps=1e-5, rope_theta=10000.0)
# (kernels, tree sizes, cached keys): digest.  one: all layers in one launch, chain: a kernel per stage, generic: the dtype-generic kernels
DIGESTS = {
    ("one", (1,), 330): "6a1f6aee04cbc2c7",
    ("one", (8,), 330): "90dfd5069ac32c00",
    ("one", (13,), 330): "d7c68775a2310169",
    ("one", (2,), 1500): "e9e20c018c50c79e",
    ("one", (16,), 2100): "9c46cd2a0a4273b6",
    ("chain", (1,), 330): "f679de54be5d451a",
    ("chain", (16,), 330): "8877651cfc79f8be",
    ("chain", (24,), 500): "0be7ddba71154ed3",
    ("chain", (37,), 330): "b79ffac7b663dd1a",
    ("chain", (64,), 900): "3f4dba1362c07abe",
    ("chain", (24, 31), 260): "7e92a8b5d8126acd",
    ("chain", (24, 31, 40), 260): "144f0922358248d8",
    ("chain", (64,) * 5, 200): "fcd53c5dec5d3b17",
    ("generic", (1,), 90): "61a8d7b8e31364a0",
    ("generic", (60,), 90): "ece40dc5e1c955fa",
    ("prefill", (40,), 0): "7fa7e7d74fe208be",
    ("prefill", (200,), 0): "28d2cf6bf89637b2",
    ("prefill", (330,), 0): "7701d03d90e0301c",
}


def _digest(*arrays):
    h = hashlib.sha256()
    for a in arrays:
        h.update(np.ascontiguousarray(a).tobytes())
    return h.hexdigest()[:16]


@pytest.fixture(scope="module")
def weights():
    made = {}

    def get(kind):
        if kind not in made:
            cfg = dict(wl.MODELS["tiny"], d_model=520, d_ffn=2056, n_heads=4, n_kv_heads=2, head_dim=32) if kind == "f32" else CLASS
            made[kind] = cfg, wl.make_weights(cfg, 1201, kind)
        return made[kind]

    return get


@pytest.mark.parametrize("path,sizes,L", [
    ("one", (1,), 330), ("one", (8,), 330), ("one", (13,), 330), ("one", (2,), 1500), ("one", (16,), 2100),
    ("chain", (1,), 330), ("chain", (16,), 330), ("chain", (24,), 500), ("chain", (37,), 330), ("chain", (64,), 900), ("chain", (24, 31), 260),
    ("chain", (24, 31, 40), 260), ("chain", (64,) * 5, 200), ("generic", (1,), 90), ("generic", (60,), 90),
])
def test_forward_bits(path, sizes, L, weights, monkeypatch):
    from paper_2507_18181_amd.runtime import Verifier
    dtype = "f32" if path == "generic" else "bf16"
    cfg, w = weights(dtype)
    if path == "chain":
        monkeypatch.setenv("SPECASR_ONE_POLLS", "0")
    nb, cap = len(sizes), L + 64
    ver = Verifier(cfg, w, dtype, max_nodes=64, capacity=cap, max_batch=nb)
    rng = np.random.default_rng([1202, L, nb])
    lens = np.asarray([L - 3 * b for b in range(nb)], np.int32)
    K, V = wl.seeded_cache(cfg, 1203, lens, cap, dtype, batch=nb)
    ver.set_cache(K, V, lens)
    trees = [wl.random_tree(rng, n, max_children=3) for n in sizes]
    toks = [rng.integers(0, cfg["vocab"], n).astype(np.int32) for n in sizes]
    fw = ver.tree_forward(toks, trees)
    assert fw["status"] == 0
    k, v = ver.get_cache()
    top = ver.tree_forward_top2(toks, trees)
    assert top["status"] == 0
    rows = [a for b, n in enumerate(sizes) for a in (fw["logits"][b, :n].cpu().numpy(), k[b, :, :, lens[b]:lens[b] + n], v[b, :, :, lens[b]:lens[b] + n],
                                                     top["top2"][b, :n].cpu().numpy(), top["prob"][b, :n].cpu().numpy())]
    ver.close()
    assert _digest(*rows) == DIGESTS[path, sizes, L]


@pytest.mark.parametrize("n", [40, 200, 330])
def test_prefill_bits(n, weights):
    from paper_2507_18181_amd.runtime import Verifier
    cfg, w = weights("bf16")
    ver = Verifier(cfg, w, "bf16", max_nodes=64, capacity=n + 8)
    tok = np.random.default_rng([1204, n]).integers(0, cfg["vocab"], n).astype(np.int32)
    out = ver.prefill([tok])
    assert out["status"] == 0
    k, v = ver.get_cache()
    ver.close()
    assert _digest(k[..., :n, :], v[..., :n, :], out["next_token"]) == DIGESTS["prefill", (n,), 0]
