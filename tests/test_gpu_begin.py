"""The first kernel of a forward on tables that do not start on 4 elements (a caller's slice of a larger tensor), and with
more metadata words than one block copies."""
import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _shifted(t):
    """The same values one element behind an aligned address."""
    flat = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    flat[1:].copy_(t.reshape(-1))
    return flat[1:].view(t.shape)


@pytest.mark.parametrize("dtype,d_model,sizes", [("f32", 24, (5,)), ("bf16", 96, (1,)), ("bf16", 1040, (33,)), ("bf16", 592, (64, 64, 40))])
def test_unaligned_tables_give_the_same_bits(dtype, d_model, sizes):
    """The same elements are read one by one instead of four at a time: every output is equal."""
    from paper_2507_18181_amd import runtime as R
    cfg = dict(wl.MODELS["tiny"], n_layers=1, d_model=d_model, d_ffn=48, n_heads=2, n_kv_heads=1, head_dim=64, vocab=40)
    w = R.upload_weights(wl.make_weights(cfg, 731, dtype))
    rng = np.random.default_rng(732)
    emb = torch.from_numpy(rng.standard_normal((len(sizes), 64, d_model)).astype(np.float32)).cuda().to(w["tok_embed"].dtype)
    toks = [rng.integers(0, 40, n).astype(np.int32) for n in sizes]
    trees = [wl.random_tree(rng, n, max_children=3) for n in sizes]
    flags = [[i % 3 == 1 for i in range(n)] for n in sizes]
    got = []
    for shift in (False, True):
        ws = dict(w, tok_embed=_shifted(w["tok_embed"]) if shift else w["tok_embed"])
        ver = R.Verifier(cfg, ws, dtype, max_nodes=64, capacity=80, max_batch=len(sizes), weights_on_device=True)
        fw = ver.tree_forward(toks, trees, embeds=_shifted(emb) if shift else emb, use_embed=flags)
        assert fw["status"] == 0
        got.append((fw["logits"].cpu(), fw["argmax"].cpu(), ver.k.cpu(), ver.v.cpu()))
        ver.close()
    for a, b in zip(*got):
        assert torch.equal(a, b)
    assert got[0][0].abs().max() > 0


@pytest.mark.parametrize("dtype,d_model", [("f32", 24), ("f32", 1024), ("bf16", 96)])
@pytest.mark.parametrize("shift", [1, 2, 3])
def test_unaligned_gains_on_the_generic_path(dtype, d_model, shift):
    """Gains one to three elements behind an aligned address, fp32 and bf16 without repacked weights: such rows are normalised
    by the kernel of wide models instead of by the linears, equal but for the order of the sum of squares."""
    from paper_2507_18181_amd import binding as B
    from paper_2507_18181_amd import runtime as R
    cfg = dict(wl.MODELS["tiny"], n_layers=2, d_model=d_model, d_ffn=48, n_heads=2, n_kv_heads=1, head_dim=8, vocab=40)
    w = R.upload_weights(wl.make_weights(cfg, 733, dtype))
    rng = np.random.default_rng(734)
    toks, trees = [rng.integers(0, 40, 11).astype(np.int32)], [wl.random_tree(rng, 11, max_children=3)]

    def moved(g):
        flat = torch.empty(g.numel() + shift, dtype=g.dtype, device=g.device)
        flat[shift:].copy_(g)
        return flat[shift:]

    got = []
    for weights in (w, dict(w, final_norm=moved(w["final_norm"]),
                            layers=[dict(l, attn_norm=moved(l["attn_norm"]), ffn_norm=moved(l["ffn_norm"])) for l in w["layers"]])):
        ver = R.Verifier(cfg, weights, dtype, max_nodes=64, capacity=80, flags=B.SPECASR_FLAG_NO_REPACK, weights_on_device=True)
        fw = ver.tree_forward(toks, trees)
        assert fw["status"] == 0
        got.append(fw["logits"][0, :11].double().cpu())
        ver.close()
    # fp32 throughout; in bf16 a K or V element may round the other way, one step of 2^-8
    assert (got[0] - got[1]).norm() <= (1e-5 if dtype == "f32" else 4e-3) * got[0].norm()
    assert got[0].abs().max() > 0
