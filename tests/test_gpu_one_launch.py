"""Forwards of up to 16 rows of one sequence, whose layers are one launch: against the oracle and against the chain of kernels, at the
edges of its row, key and shape ranges; replayed as a graph; and what happens when a wait inside it runs out."""
import numpy as np
import pytest

import oracle
import workload as wl
from parity_util import TOL_BF16, check_forward, check_tree_kv

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = {
    "tiny": dict(n_layers=2, d_model=256, n_heads=4, n_kv_heads=4, d_ffn=672),      # 8 stages of k over 8 wavefronts, ragged half-bands
    "odd": dict(n_layers=3, d_model=608, n_heads=6, n_kv_heads=2, d_ffn=1184),      # wavefronts with 1 and 2 .. 5 stages
    "small": dict(n_layers=2, d_model=128, n_heads=2, n_kv_heads=1, d_ffn=160),     # wavefronts without any
    "grouped": dict(n_layers=2, d_model=512, n_heads=16, n_kv_heads=2, d_ffn=992),  # 8 query heads per KV head
    "wide": dict(n_layers=2, d_model=2048, n_heads=32, n_kv_heads=4, d_ffn=5632),   # the largest
}


def _cfg(shape):
    return dict(wl.MODELS["tiny"], head_dim=64, vocab=96, **SHAPES[shape])


def _verifier(cfg, w, cap, batch=1):
    from paper_2507_18181_amd.runtime import Verifier
    return Verifier(cfg, w, "bf16", max_nodes=32, capacity=cap, max_batch=batch)


def _one(err):
    return "one launch" in err


@pytest.mark.parametrize("shape,n,L", [
    ("tiny", 1, 0), ("tiny", 2, 1), ("tiny", 8, 31), ("tiny", 9, 32), ("tiny", 16, 33), ("tiny", 16, 260), ("tiny", 5, 2048), ("tiny", 16, 2050),
    ("tiny", 1, 1190), ("tiny", 3, 4096), ("odd", 1, 40), ("odd", 4, 300), ("odd", 7, 0), ("odd", 12, 97), ("odd", 16, 1), ("small", 6, 20),
    ("small", 11, 64), ("wide", 1, 30), ("wide", 8, 70), ("wide", 16, 15),
])
def test_against_the_oracle_and_the_chain(shape, n, L, monkeypatch, capfd):
    cfg = _cfg(shape)
    w = wl.make_weights(cfg, 911, "bf16")
    rng = np.random.default_rng([912, n, L])
    cap = L + n + 3
    K, V = wl.seeded_cache(cfg, 913, np.asarray([L], np.int32), cap, "bf16", batch=1)
    tree = wl.random_tree(rng, n, max_children=3)
    tok = rng.integers(0, cfg["vocab"], n).astype(np.int32)
    ref = oracle.OracleModel(cfg, w).tree_forward(np.ascontiguousarray(K[0]), np.ascontiguousarray(V[0]), L, tok, tree)
    monkeypatch.setenv("SPECASR_DEBUG", "1")
    got = []
    for polls in (None, "0"):
        if polls:
            monkeypatch.setenv("SPECASR_ONE_POLLS", polls)
        ver = _verifier(cfg, w, cap)
        ver.set_cache(K, V, [L])
        capfd.readouterr()
        fw = ver.tree_forward([tok], [tree])
        assert fw["status"] == 0
        assert _one(capfd.readouterr().err) == (polls is None)
        k1, v1 = ver.get_cache()
        lg = fw["logits"][0].cpu().numpy()
        check_forward(ref, lg, fw["argmax"][0].cpu().numpy(), TOL_BF16)
        check_tree_kv(k1[0], v1[0], L, ref, TOL_BF16)
        if polls is None:  # the same bits again: every sum has one order
            fw = ver.tree_forward([tok], [tree])
            k2, v2 = ver.get_cache()
            assert np.array_equal(lg, fw["logits"][0].cpu().numpy()) and np.array_equal(k1, k2) and np.array_equal(v1, v2)
        got.append(lg[:n].astype(np.float64))
        ver.close()
    # two orders of fp32 sums and, behind them, single K and V elements that round the other way (a step of 2^-8 of an element)
    assert np.linalg.norm(got[0] - got[1]) <= 2.5e-3 * np.linalg.norm(got[1])


@pytest.mark.parametrize("n,batch,L,layers", [(17, 1, 20, 2), (4, 2, 20, 2), (4, 1, 4097, 2), (4, 1, 20, 1)])
def test_what_stays_on_the_chain(n, batch, L, layers, monkeypatch, capfd):
    cfg = dict(_cfg("tiny"), n_layers=layers)
    w = wl.make_weights(cfg, 921, "bf16")
    monkeypatch.setenv("SPECASR_DEBUG", "1")
    ver = _verifier(cfg, w, L + n, batch)
    ver.kv_len[:] = L
    capfd.readouterr()
    fw = ver.tree_forward([np.arange(n, dtype=np.int32)] * batch, [np.arange(-1, n - 1, dtype=np.int32)] * batch)
    err = capfd.readouterr().err
    assert fw["status"] == 0 and "plan qkv" in err and not _one(err)
    ver.close()


def test_whole_rounds_and_input_rows():
    """verify_tree and the draft-side read-out on this path, with embedding rows among the inputs, against the chain."""
    import os
    cfg = _cfg("odd")
    w = wl.make_weights(cfg, 931, "bf16")
    rng = np.random.default_rng(932)
    n, L, cap = 13, 50, 96
    K, V = wl.seeded_cache(cfg, 933, np.asarray([L], np.int32), cap, "bf16", batch=1)
    tree = wl.random_tree(rng, n, max_children=2)
    tok = rng.integers(0, cfg["vocab"], n).astype(np.int32)
    emb = torch.from_numpy(rng.standard_normal((1, 32, cfg["d_model"])).astype(np.float32)).to("cuda:0").to(torch.bfloat16)
    outs = []
    for polls in (None, "0"):
        if polls:
            os.environ["SPECASR_ONE_POLLS"] = polls
        try:
            ver = _verifier(cfg, w, cap)
        finally:
            os.environ.pop("SPECASR_ONE_POLLS", None)
        ver.set_cache(K, V, [L])
        top = ver.tree_forward_top2([tok], [tree], want_logits=True, embeds=emb, use_embed=[[i % 3 == 0 for i in range(n)]])
        vt = ver.verify_tree([tok], [tree], want_logits=True)
        assert top["status"] == 0 and vt["status"] == 0
        outs.append((top["logits"][0, :n].double().cpu().numpy(), vt["logits"][0, :n].double().cpu().numpy(), vt["accept_len"][0], int(ver.kv_len[0])))
        ver.close()
    for a, b in ((outs[0][0], outs[1][0]), (outs[0][1], outs[1][1])):
        assert np.linalg.norm(a - b) <= 2.5e-3 * np.linalg.norm(b)
    assert outs[0][2:] == outs[1][2:]


def test_replayed_as_a_graph():
    """The launch counts its items in scratch that the first kernel of the call clears: replays give the eager bits."""
    from paper_2507_18181_amd import binding as B
    cfg = _cfg("tiny")
    w = wl.make_weights(cfg, 941, "bf16")
    rng = np.random.default_rng(942)
    n, L = 10, 40
    K, V = wl.seeded_cache(cfg, 943, np.asarray([L], np.int32), 64, "bf16", batch=1)
    tree = wl.random_tree(rng, n, max_children=3)
    tok = rng.integers(0, cfg["vocab"], n).astype(np.int32)
    ver = _verifier(cfg, w, 64)
    ver.set_cache(K, V, [L])
    eager = ver.tree_forward([tok], [tree])["logits"].clone()
    argmax = torch.full((1, 32), -1, dtype=torch.int32, device="cuda:0")
    logits = torch.zeros((1, 32, cfg["vocab"]), device="cuda:0")
    t, keep = ver._tree([tok], [tree])
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        assert B.specasr_tree_forward(ver.ctx, ver._kv, t, argmax, logits, ver.ws_ptr, ver.ws_bytes, s.cuda_stream) == 0
    for _ in range(4):
        logits.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(logits, eager)
    ver.close()


def test_a_wait_that_runs_out_is_reported(monkeypatch):
    """With a bound of a single look every wait is given up at once: the launch ends all the same, and the call says so."""
    from paper_2507_18181_amd import binding as B
    cfg = _cfg("tiny")
    w = wl.make_weights(cfg, 951, "bf16")
    monkeypatch.setenv("SPECASR_ONE_POLLS", "1")
    ver = _verifier(cfg, w, 64)
    ver.kv_len[:] = 20
    out = ver.verify_tree([np.arange(9, dtype=np.int32)], [np.arange(-1, 8, dtype=np.int32)])
    assert out["status"] == B.SPECASR_E_HIP and ver.kv_len[0] == 20
    ver.close()


@pytest.mark.parametrize("what", ["embedding", "input row", "key", "value", "infinite key", "gain", "weight row"])
@pytest.mark.parametrize("shape,n,L", [("odd", 7, 40), ("tiny", 12, 2090)])
def test_nan_and_infinity_as_in_the_chain(shape, n, L, what, monkeypatch):
    """All ones, a NaN in float and in bf16, stands for missing data between the workgroups of the launch and may be data all the same.  A value that a
    reader would wait for in vain gives up after 20000 looks (the status says so) instead of 2 million."""
    cfg = _cfg(shape)
    w = wl.make_weights(cfg, 961, "bf16")
    rng = np.random.default_rng([962, n])
    cap = L + n
    K, V = wl.seeded_cache(cfg, 963, np.asarray([L], np.int32), cap, "bf16", batch=1)
    tok = np.arange(n, dtype=np.int32)
    tree = wl.random_tree(rng, n, max_children=3)
    emb, use = None, None
    if what == "embedding":
        w["tok_embed"][tok[n - 1]] = 0xffff
    elif what == "input row":
        emb = torch.full((1, 32, cfg["d_model"]), -1, dtype=torch.int16, device="cuda:0").view(torch.bfloat16)
        use = [[i == n // 2 for i in range(n)]]
    elif what == "key":
        K[0, 1, 0, L // 2] = 0xffff
    elif what == "value":
        V[0, 0, -1, L - 1] = 0xffff
    elif what == "infinite key":
        K[0, 1, 0, 3, 5] = 0x7f80
    elif what == "gain":
        w["layers"][1]["ffn_norm"][-3:] = 0xffff
    else:
        w["layers"][0]["wv"][1] = 0xffff
        w["layers"][1]["w_up"][-1] = 0xffff
    got = []
    for polls in ("20000", "0"):
        monkeypatch.setenv("SPECASR_ONE_POLLS", polls)
        ver = _verifier(cfg, w, cap)
        ver.set_cache(K, V, [L])
        fw = ver.tree_forward([tok], [tree], embeds=emb, use_embed=use)
        again = ver.verify_tree([tok], [tree]) if emb is None else fw  # synchronises: reports a wait that ran out
        assert fw["status"] == 0 and again["status"] == 0
        k1, v1 = ver.get_cache()
        got.append([fw["logits"][0, :n].double().cpu().numpy()] + [wl.bf16_to_f32(c[..., L:L + n, :]).astype(np.float64) for c in (k1, v1)])
        ver.close()
    assert any(np.isnan(a).any() for a in got[1])
    for a, b in zip(*got):
        assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isinf(a), np.isinf(b))
        ok = np.isfinite(b)
        # the bound of two orders of fp32 sums, as above, over what is finite
        assert np.linalg.norm(a[ok] - b[ok]) <= 2.5e-3 * max(np.linalg.norm(b[ok]), 1e-30)


def _gives_up(monkeypatch, looks="1"):
    cfg = _cfg("tiny")
    monkeypatch.setenv("SPECASR_ONE_POLLS", looks)
    ver = _verifier(cfg, wl.make_weights(cfg, 951, "bf16"), 64)
    K, V = wl.seeded_cache(cfg, 952, np.asarray([20], np.int32), 64, "bf16", batch=1)
    ver.set_cache(K, V, [20])
    return ver, np.arange(9, dtype=np.int32), np.arange(-1, 8, dtype=np.int32)


@pytest.mark.parametrize("call", ["tree_forward", "tree_forward_top2"])
def test_a_forward_that_gave_up_is_not_handed_on(call, monkeypatch):
    """The wrappers wait for the forward, so its own status says that it is void."""
    from paper_2507_18181_amd import binding as B
    ver, tok, par = _gives_up(monkeypatch)
    assert getattr(ver, call)([tok], [par])["status"] == B.SPECASR_E_HIP
    ver.close()


@pytest.mark.parametrize("replay", [False, True])
def test_a_forward_that_gave_up_is_not_committed(replay, monkeypatch):
    """An asynchronous forward, eager or replayed: told after the synchronisation, and nothing that follows accepts or commits it, on this stream
    or another, however often it is asked."""
    from paper_2507_18181_amd import binding as B
    ver, tok, par = _gives_up(monkeypatch)
    argmax = torch.full((1, 32), -1, dtype=torch.int32, device="cuda:0")
    logits = torch.zeros((1, 32, ver.cfg["vocab"]), device="cuda:0")
    t, keep = ver._tree([tok], [par])
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()

    def forward():
        return B.specasr_tree_forward(ver.ctx, ver._kv, t, argmax, logits, ver.ws_ptr, ver.ws_bytes, s.cuda_stream)

    assert ver.accept([tok], [par], argmax_dev=argmax)["status"] == B.SPECASR_OK  # pinned memory is there: nothing is allocated under capture
    if replay:
        with torch.cuda.graph(g, stream=s):
            assert forward() == B.SPECASR_OK
        assert B.specasr_last_hip_error(ver.ctx) == 0
        g.replay()
    else:
        assert forward() == B.SPECASR_OK
    torch.cuda.synchronize()
    assert B.specasr_last_hip_error(ver.ctx) == B.HIP_ERROR_LAUNCH_TIMEOUT
    assert torch.isnan(logits[0, :9]).any()  # computed from what was missing
    before = ver.get_cache()
    for _ in range(2):
        assert ver.commit([9], [[0, 2, 4]]) == B.SPECASR_E_HIP
        assert ver.verify_tree([tok], [par])["status"] == B.SPECASR_E_HIP
        assert ver.accept([tok], [par], argmax_dev=argmax)["status"] == B.SPECASR_E_HIP
        assert ver.accept([tok], [par], logits_dev=logits)["status"] == B.SPECASR_E_HIP
        assert ver.prefill([tok])["status"] == B.SPECASR_E_HIP
        out = [torch.zeros(32, dtype=torch.int32, device="cuda:0") for _ in range(4)]
        assert B.specasr_accept_from_logits_static(ver.ctx, t, 1, logits, *out, None) == B.SPECASR_E_HIP
        assert B.specasr_last_hip_error(ver.ctx) == B.HIP_ERROR_LAUNCH_TIMEOUT
    assert ver.kv_len[0] == 20
    assert all(np.array_equal(a, b) for a, b in zip(before, ver.get_cache()))
    ver.close()


def test_workspace(monkeypatch):
    """The launch has its scratch where wide passes have theirs: as long as it fits, no call needs a larger workspace for it; without wide
    passes a workspace for one sequence grows by it, and one for several sequences also serves calls of one."""
    from paper_2507_18181_amd import binding as B
    from paper_2507_18181_amd.runtime import Verifier
    cfg = _cfg("wide")
    w = wl.make_weights(cfg, 971, "bf16")
    sizes = {}
    for polls in (None, "0"):
        if polls:
            monkeypatch.setenv("SPECASR_ONE_POLLS", polls)
        for flags in (0, B.SPECASR_FLAG_NO_WIDE):
            ver = Verifier(cfg, w, "bf16", max_nodes=32, capacity=64, max_batch=16, flags=flags)
            sizes[polls, flags] = [B.specasr_workspace_bytes(ver.ctx, b) for b in (1, 2, 16)]
            ver.close()
    assert sizes[None, 0] == sizes["0", 0]
    one, chain = sizes[None, B.SPECASR_FLAG_NO_WIDE], sizes["0", B.SPECASR_FLAG_NO_WIDE]
    assert one[0] > chain[0] and one == sorted(one) and one[2] == chain[2]


@pytest.mark.parametrize("call", ["tree_forward", "tree_forward_top2", "verify_tree"])
def test_workspace_that_only_holds_the_chain(call, monkeypatch):
    """What a call needs without the launch is still enough for it: it runs as the chain, whose bits it gives; one byte less is refused."""
    from paper_2507_18181_amd import binding as B
    from paper_2507_18181_amd.runtime import Verifier
    cfg = _cfg("wide")
    w = wl.make_weights(cfg, 971, "bf16")
    K, V = wl.seeded_cache(cfg, 972, np.asarray([20], np.int32), 64, "bf16", batch=1)
    tok, par = np.arange(9, dtype=np.int32), np.arange(-1, 8, dtype=np.int32)
    monkeypatch.setenv("SPECASR_ONE_POLLS", "0")
    res, size = [], None
    for chain in (True, False):
        if not chain:
            monkeypatch.delenv("SPECASR_ONE_POLLS")
        ver = Verifier(cfg, w, "bf16", max_nodes=32, capacity=64, flags=B.SPECASR_FLAG_NO_WIDE)
        ver.set_cache(K, V, [20])
        if chain:
            size = ver.ws_bytes
        assert size <= ver.ws_bytes and chain == (size == ver.ws_bytes)
        ver.ws_bytes = size
        out = getattr(ver, call)([tok], [par], want_logits=True)
        assert out["status"] == 0
        res.append([out["logits"].cpu().numpy()] + list(ver.get_cache()))
        ver.ws_bytes = size - 1
        ver.kv_len[0] = 20
        assert getattr(ver, call)([tok], [par])["status"] == B.SPECASR_E_WORKSPACE
        ver.close()
    assert all(np.array_equal(a, b) for a, b in zip(*res))


@pytest.mark.parametrize("wide", [True, False])
def test_between_passes_over_many_rows(wide, monkeypatch):
    """Prefill, a forward in one launch and prefill again, enqueued one behind the other in one workspace, against contexts of their own."""
    from paper_2507_18181_amd import binding as B
    from paper_2507_18181_amd.runtime import Verifier
    cfg = _cfg("odd")
    w = wl.make_weights(cfg, 981, "bf16")
    rng = np.random.default_rng(982)
    first, second, tok = (rng.integers(0, cfg["vocab"], n).astype(np.int32) for n in (90, 70, 11))
    par = wl.random_tree(rng, 11, max_children=3)
    flags = 0 if wide else B.SPECASR_FLAG_NO_WIDE

    def run(calls):
        ver = Verifier(cfg, w, "bf16", max_nodes=32, capacity=256, flags=flags)
        argmax = torch.full((1, 32), -1, dtype=torch.int32, device="cuda:0")
        logits = torch.zeros((1, 32, cfg["vocab"]), device="cuda:0")
        for what in calls:
            if isinstance(what, str):
                t, keep = ver._tree([tok], [par])
                assert B.specasr_tree_forward(ver.ctx, ver._kv, t, argmax, logits, ver.ws_ptr, ver.ws_bytes, None) == 0
            else:
                n = np.asarray([len(what)], np.int32)
                assert B.specasr_prefill(ver.ctx, ver._kv, what[None], None, None, n, len(what), None, ver.ws_ptr, ver.ws_bytes, None) == 0
        torch.cuda.synchronize()
        out = logits.cpu().numpy(), [c[..., :ver.kv_len[0], :] for c in ver.get_cache()]
        ver.close()
        return out

    mixed = run([first, "tree", second, "tree", first])
    prefills = run([first, second, first])
    assert all(np.array_equal(a, b) for a, b in zip(mixed[1], prefills[1]))
    assert np.array_equal(mixed[0], run([first, second, "tree"])[0])


@pytest.mark.parametrize("n,L,groups,chunks", [(1, 1200, 1, 3), (2, 4096, 1, 8), (4, 1152, 1, 1), (4, 1153, 1, 3), (5, 1153, 2, 1), (5, 2048, 2, 1), (5, 2100, 2, 5), (8, 4096, 2, 8), (9, 2100, 3, 5), (16, 2100, 4, 5), (16, 4096, 4, 8)])
def test_groups_of_query_rows_and_chunks_of_keys(n, L, groups, chunks, monkeypatch, capfd):
    """Several of both: which partial output is whose.  The number of chunks is the plan's own, so that another rule cannot leave this without any."""
    assert groups == (8 * n + 31) // 32
    test_against_the_oracle_and_the_chain("grouped", n, L, monkeypatch, capfd)
    monkeypatch.delenv("SPECASR_ONE_POLLS")
    cfg = _cfg("grouped")
    ver = _verifier(cfg, wl.make_weights(cfg, 911, "bf16"), L + n)
    ver.kv_len[:] = L
    capfd.readouterr()
    assert ver.tree_forward([np.arange(n, dtype=np.int32)], [np.arange(-1, n - 1, dtype=np.int32)])["status"] == 0
    assert "%d key chunks" % chunks in capfd.readouterr().err
    ver.close()


@pytest.mark.parametrize("shift", [1, 4])
@pytest.mark.parametrize("n,L", [(8, 300), (8, 2100), (13, 300), (16, 2100)])
def test_cache_that_is_not_on_16_bytes(n, L, shift):
    """K and V 2 or 8 bytes into a larger tensor, read through registers: the bits of an aligned cache, up to 8 rows and beyond."""
    from paper_2507_18181_amd import binding as B
    cfg = _cfg("grouped")
    w = wl.make_weights(cfg, 991, "bf16")
    rng = np.random.default_rng([992, n, L])
    cap = L + n + 5
    K, V = wl.seeded_cache(cfg, 993, np.asarray([L], np.int32), cap, "bf16", batch=1)
    tree = wl.random_tree(rng, n, max_children=3)
    tok = rng.integers(0, cfg["vocab"], n).astype(np.int32)
    res = []
    for s in (0, shift):
        ver = _verifier(cfg, w, cap)
        ver.k, ver.v = (torch.zeros(t.numel() + s, dtype=t.dtype, device=t.device)[s:].view(t.shape) for t in (ver.k, ver.v))
        assert ver.k.data_ptr() % 16 == ver.v.data_ptr() % 16 == 2 * s
        ver._kv = B.make_kv(ver.k, ver.v, cap, ver.kv_len)
        ver.set_cache(K, V, [L])
        fw = ver.tree_forward([tok], [tree])
        vt = ver.verify_tree([tok], [tree], want_logits=True)
        assert fw["status"] == 0 and vt["status"] == 0
        res.append([fw["logits"].cpu().numpy(), vt["logits"].cpu().numpy(), vt["path"]] + list(ver.get_cache()))
        ver.close()
    for a, b in zip(*res):
        assert np.array_equal(a, b)


def test_few_heads_are_cut_early(monkeypatch, capfd):
    """Up to 64 rows of heads the partial outputs are few: chunks from 37 tiles of 32 keys on, also with 16 rows (2000 keys of one KV head in one chunk took longer
    than the chain of kernels)."""
    test_against_the_oracle_and_the_chain("small", 16, 2000, monkeypatch, capfd)
    monkeypatch.delenv("SPECASR_ONE_POLLS")
    cfg = _cfg("small")
    ver = _verifier(cfg, wl.make_weights(cfg, 911, "bf16"), 2016)
    ver.kv_len[:] = 2000
    capfd.readouterr()
    assert ver.tree_forward([np.arange(16, dtype=np.int32)], [np.arange(-1, 15, dtype=np.int32)])["status"] == 0
    assert "4 key chunks" in capfd.readouterr().err
    ver.close()
