"""How far the fp32 sums of the half-band GEMM's feed-forward projections are from 64 bits with 1 .. 8 rows, where one
operand holds both activation planes."""
import re

import numpy as np
import pytest

import workload as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

D_SMALL = 2.0 ** -30   # scale of the embedding rows: far below the sums' errors, which are then what the forward returns


def _forward(cfg, w, n, capfd):
    """Residual rows behind the only layer: the last norm's rms is that of eps alone and lm_head is the identity."""
    from paper_2507_18181_amd.runtime import Verifier
    ver = Verifier(cfg, w, "bf16", max_nodes=8, capacity=16)
    capfd.readouterr()
    fw = ver.tree_forward([np.arange(n, dtype=np.int32)], [np.arange(-1, n - 1, dtype=np.int32)])
    assert fw["status"] == 0
    plan = dict(re.findall(r"plan (\w+) rows=%d .*: (.+?), \d+ splits" % n, capfd.readouterr().err))
    got = fw["logits"][0, :n].double().cpu().numpy() * np.sqrt(cfg["rms_eps"])
    ver.close()
    return got, plan


def _weights(cfg, rng, gate, up, down, order):
    d, F, dq, dkv = cfg["d_model"], cfg["d_ffn"], 128, 64
    one = np.ones(d, np.float32)
    gain = 1.0 + 0.2 * rng.standard_normal(d).astype(np.float32)   # the normalised rows need both planes
    gain[d // 2:] = gain[:d // 2]
    gain = gain[order]
    zero = lambda *s: np.zeros(s, np.float32)
    emb = rng.standard_normal((cfg["vocab"], d)).astype(np.float32) * D_SMALL
    emb[:, d // 2:] = emb[:, :d // 2]
    emb = emb[:, order]
    layer = dict(attn_norm=one, wq=zero(dq, d), wk=zero(dkv, d), wv=zero(dkv, d), wo=zero(d, dq), ffn_norm=gain, w_gate=gate, w_up=up, w_down=down)
    w = dict(tok_embed=emb, final_norm=one, lm_head=np.eye(d, dtype=np.float32), layers=[layer])
    return {k: wl.bf16_bits(v) if k != "layers" else [{n: wl.bf16_bits(m) for n, m in v[0].items()}] for k, v in w.items()}


# rms errors in units of 2^-24 of the rms that the whole sum would have.  One rounding (to nearest, of a sum whose leading digit
# is anywhere) has an rms of 0.42; a step of 32 products rounds 4 times.  A slice of L steps whose products run in chains
# contributes 0.72 per step times the running length, an addition of sums 0.18 times the length so far, both over L:
#                                                  blocks of 4 (2)     chains over the slice
#   13B down, slices of 18 steps in 3 splits          1.7 (1.64)           2.1 (2.04)     two chains
#   gate|up of 8192 features, slices of 16            1.5 (1.30)           1.7 (1.57)     two chains
#   gate|up of 16384 features, slices of 16           1.4 (1.24)           2.4 (2.04)     one chain
# with the additions over slices and splits; measured in brackets.  The bounds stand in the middle of what is measured.
@pytest.mark.parametrize("stage,kernel,d,F,bound", [
    ("down", "slice 4x0", 5120, 13824, 1.83),
    ("gate_up", "slice 4x0", 4096, 8192, 1.43),
    ("gate_up", "slice 8x0", 4096, 16384, 1.63),
])
def test_feed_forward_chains_of_few_rows(stage, kernel, d, F, bound, monkeypatch, capfd):
    """Every product of a sum has its negative somewhere else in k, so the exact sum is zero and what comes out is the
    rounding of the sums alone; equal features have equal bits, so nothing in front of the sum adds to it."""
    monkeypatch.setenv("SPECASR_DEBUG", "1")
    rng = np.random.default_rng(771)
    n = 8
    cfg = dict(wl.MODELS["tiny"], n_layers=1, d_model=d, d_ffn=F, n_heads=2, n_kv_heads=1, head_dim=64, vocab=d)
    scale = np.float32(np.sqrt(cfg["rms_eps"]) / D_SMALL / np.sqrt(d))   # a product of a whole row of k is about 1
    gate = rng.standard_normal((F, d), dtype=np.float32) * scale
    up = rng.standard_normal((F, d), dtype=np.float32) * scale
    down = np.zeros((d, F), np.float32)
    order = rng.permutation(d)
    if stage == "down":
        gate[F // 2:], up[F // 2:] = gate[:F // 2], up[:F // 2]
        down[:] = rng.standard_normal((d, F), dtype=np.float32)
        down[:, F // 2:] = -down[:, :F // 2]
        at = rng.permutation(F)
        gate, up, down = gate[at], up[at], down[:, at]
    else:
        gate[:, d // 2:] = -gate[:, :d // 2]
        gate = gate[:, order]
        down[np.arange(d), np.arange(d) * (F // d)] = 1.0   # output i shows feature i * F / d
    w = _weights(cfg, rng, gate, up, down, order)
    got, plan = _forward(cfg, w, n, capfd)
    assert plan[stage] == kernel, plan
    x = wl.bf16_to_f32(w["tok_embed"]).astype(np.float64)[:n]
    err = got - x
    lw = w["layers"][0]
    h = x / np.sqrt((x * x).mean(1, keepdims=True) + cfg["rms_eps"]) * wl.bf16_to_f32(lw["ffn_norm"])
    f64 = lambda k: torch.from_numpy(wl.bf16_to_f32(lw[k])).double()
    g, u = (torch.from_numpy(h) @ f64(k).t() for k in ("w_gate", "w_up"))
    if stage == "down":
        t = (g * torch.sigmoid(g) * u).numpy()
        unit = np.sqrt((t * t).sum(1, keepdims=True)) * np.sqrt((f64("w_down") ** 2).mean().item())
    else:
        # silu(e) * u is e * u / 2 for the small e that is left of the gate
        err = 2.0 * err / u.numpy()[:, ::F // d][:, :d]
        keep = np.abs(u.numpy()[:, ::F // d][:, :d]) > 0.3   # smaller ones bring the residual's own bits in
        err = np.where(keep, err, 0.0)
        unit = np.sqrt((h * h).sum(1, keepdims=True)) * np.sqrt((f64("w_gate") ** 2).mean().item()) * np.sqrt(keep.mean())
    rel = np.sqrt(((err / unit) ** 2).mean()) * 2.0 ** 24
    print("%s %d x %d: %.3f units of 2^-24" % (stage, d, F, rel))
    assert rel <= bound
