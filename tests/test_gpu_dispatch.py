"""Edges of the kernels' size ranges and of the rules that choose between them (GPU)."""
import numpy as np
import pytest
import torch

import parity as P
import workloads as wl

pytestmark = pytest.mark.gpu

FIELDS = ("H", "s", "win_k", "win_v", "sp_k", "sp_v", "sp_idx", "sp_count", "n_tokens")


@pytest.mark.parametrize("B,Hkv,d,D,eta,lam,kw", [(1, 1, 32, 2, 1, 1, {}), (3, 1, 64, 6, 5, 0, {}), (1, 3, 128, 128, 64, 128, dict(fold_defer=8)),
                                                  (2, 5, 64, 64, 16, 33, dict(score_kind=1)), (9, 7, 128, 256, 0, 257, {})])
def test_reset_empties_every_field(B, Hkv, d, D, eta, lam, kw):
    """One launch fills all fields: word counts that are no multiple of four or of a block's share, fields of no words,
    the optional ones; nothing outside the fields is written (guard words behind each)."""
    from paper_2505_23666_amd import binding as lb
    lay = lb.LolaLayer(B, Hkv, Hkv, d, D, eta, lam, 16, dtype="bf16", **kw)
    names = FIELDS + (("pend_phi", "pend_v", "pend_count") if kw.get("fold_defer") else ()) + (("win_score", "sp_score") if kw.get("score_kind") else ())
    bufs = {}
    for n in names:
        t = getattr(lay, n)
        raw = torch.full((t.numel() * t.element_size() + 64,), 0x5A, dtype=torch.uint8, device=P.DEV)
        bufs[n] = (raw, t.numel() * t.element_size())
        if t.numel():
            setattr(lay.st, n, raw.data_ptr())
    lb.lola_state_init(lay.cfg, lay.st)
    torch.cuda.synchronize()
    for n, (raw, nb) in bufs.items():
        want = 0xFF if n == "sp_idx" else 0
        assert bool((raw[:nb] == want).all()), n
        assert bool((raw[nb:] == 0x5A).all()), n


def test_reset_of_more_memories_than_a_grid_of_blocks():
    """Fields that together pass 256 GiB need more than one launch grid of the usual blocks.  The four K / V fields (64 GiB each)
    share one buffer here."""
    from paper_2505_23666_amd import binding as lb
    ns, d, D, rows = 16400, 256, 2, 4096
    cfg = lb.LolaConfig(ns, 1, 1, d, D, rows, rows, 16, lb.LOLA_F32, lb.LOLA_F32, 0, 0.0, 0, 0, 0, 0)
    tot, fb = lb.lola_state_bytes(cfg)
    assert tot >> 38 and fb[2] == fb[3] == fb[4] == fb[5]
    torch.cuda.empty_cache()
    size = {0: fb[0], 1: fb[1], 2: fb[2], 6: fb[6], 7: fb[7], 8: fb[8]}
    bufs = {i: torch.full((n + 64,), 0x5A, dtype=torch.uint8, device=P.DEV) for i, n in size.items()}
    st = lb.LolaState(*[bufs[2 if 2 <= i <= 5 else i].data_ptr() if i < 9 else None for i in range(14)])
    lb.lola_state_init(cfg, st)
    torch.cuda.synchronize()
    for i, n in size.items():
        raw, want = bufs[i], 0xFF if i == 6 else 0
        for a in range(0, n, 1 << 30):
            assert bool((raw[a:min(n, a + (1 << 30))] == want).all()), (i, a)
        assert bool((raw[n:] == 0x5A).all()), i
    del bufs, raw
    torch.cuda.empty_cache()


def case_inputs(seed, B, Hq, Hkv, d, D, N, wscale=1.0):
    g = wl.rng(seed, 5)
    mk = lambda *shape: wl.store(g.standard_normal(shape, dtype=np.float32), "bf16")
    w = lambda H: wl.store((wscale * g.standard_normal((H, d, D // 2), dtype=np.float32) / np.sqrt(d)).astype(np.float32), "bf16")
    return mk(B, Hq, N, d), mk(B, Hkv, N, d), mk(B, Hkv, N, d), w(Hq), w(Hkv)


@pytest.mark.parametrize("d,D,eta,lam,kw", [(128, 128, 64, 128, {}), (64, 128, 64, 64, {}), (128, 128, 64, 256, {}),
                                            (64, 128, 64, 256, {}), (128, 256, 128, 192, {}), (64, 256, 192, 64, dict(phi_kind=1)),
                                            (128, 128, 128, 0, {}), (64, 256, 192, 0, {}), (128, 128, 64, 128, dict(score_kind=4)),
                                            (128, 256, 64, 128, dict(score_kind=1))])
def test_calls_that_end_while_window_and_cache_fill(d, D, eta, lam, kw):
    """Calls of every awkward length before, across and behind the point where window and cache are full: their filling
    chunks are copied in one go, the first scored chunk may find an incomplete cache, a ragged last one folds fewer than
    64 pairs; every third call in one-chunk workspace passes.  Outputs, memories and every chunk's selection against the
    oracle, then the same without outputs."""
    full = eta + lam
    lens = [1, 62, 2, 65, 30, max(1, full - 170), 11, 64, 129, 3, 200]
    cuts = np.concatenate([[0], np.cumsum(lens)])
    sh = wl.Shape("fill", "bf16", 2, 4, 2, d, D, T=0, eta=eta, lam=lam, C=64, seed=0)
    q, k, v, Wq, Wk = case_inputs(40 + d + D + eta + lam, 2, 4, 2, d, D, int(cuts[-1]), wscale=0.5 if kw.get("phi_kind") else 1.0)
    for outputs in (True, False):
        if not outputs and kw.get("score_kind"):
            continue
        layer, o = None, None
        for i, (a, b) in enumerate(zip(cuts, cuts[1:])):
            print("fill", d, D, eta, lam, kw, "call", i, int(a), int(b), "outputs", outputs, flush=True)
            layer, o, rep = P.prefill_parity(sh, q[:, :, a:b], k[:, :, a:b], v[:, :, a:b], Wq, Wk, layer=layer, oracle=o, layer_kw=kw,
                                             with_outputs=outputs, workspace_limit=0 if i % 3 == 2 else None)
            assert layer.lola_path[0] == "mfma"
        assert rep["scored"] > 0 or lam == 0
    # one call from empty memories that crosses the point, in one-chunk passes: the filling chunks of later passes too
    for T in (full + 64 + 5, max(64, full - 3)):
        P.prefill_parity(sh, q[:, :, :T], k[:, :, :T], v[:, :, :T], Wq, Wk, layer_kw=kw, workspace_limit=0)


IRREGULAR = [(128, 128, 64, 128, {}), (64, 128, 64, 64, {}), (128, 128, 64, 64, {}), (128, 128, 64, 256, {}), (64, 128, 64, 256, {}), (128, 256, 128, 128, {}),
             (64, 256, 64, 512, {}), (128, 128, 128, 64, {}), (64, 128, 128, 192, {}), (128, 128, 64, 128, dict(phi_kind=1)), (128, 256, 128, 192, dict(phi_kind=1))]


def irregular_calls(eta, lam):
    """(first and last token of each call): one that ends 40 tokens behind the full cache, or that fills it and then 24 short ones"""
    short = [int(x) for x in wl.rng(eta + lam, 7).integers(1, 64, 24)]
    for lens in ([eta + lam + 40], [eta + lam] + short):
        cuts = np.concatenate([[0], np.cumsum(lens)])
        yield [(int(a), int(b)) for a, b in zip(cuts, cuts[1:])]


@pytest.mark.parametrize("d,D,eta,lam,kw", IRREGULAR + [(64, 256, 128, 0, {}), (128, 128, 64, 128, dict(score_kind=1))])
def test_irregular_chunks_fold_in_fp32(d, D, eta, lam, kw):
    """Chunks that fold fewer than 64 pairs (the first scored one, ragged last ones) fold fp32 features as the shape-generic
    kernels do: H and s stay within 2^-20 of the oracle, sixteen roundings of 2^-24 for the feature and the sums; features in
    two bf16 parts leave 2^-18 of each product (H off by more than 2.5e-6)."""
    sh = wl.Shape("irr", "bf16", 2, 4, 2, d, D, T=0, eta=eta, lam=lam, C=64, seed=0)
    for calls in irregular_calls(eta, lam):
        q, k, v, Wq, Wk = case_inputs(11 + d + D + lam, 2, 4, 2, d, D, calls[-1][1], wscale=0.5 if kw.get("phi_kind") else 1.0)
        layer, o = None, None
        for a, b in calls:
            print("irregular", d, D, eta, lam, kw, a, b, flush=True)
            layer, o, rep = P.prefill_parity(sh, q[:, :, a:b], k[:, :, a:b], v[:, :, a:b], Wq, Wk, layer=layer, oracle=o, layer_kw=kw)
        assert layer.lola_path[0] == "mfma" and rep["scored"] > 0 or lam == 0
        assert rep["H_err"] < 2.0 ** -20 and rep["s_err"] < 2.0 ** -20, (rep["H_err"], rep["s_err"])


@pytest.mark.parametrize("d,D,eta,lam,kw", IRREGULAR)
def test_irregular_chunks_rank_close_recalls(d, D, eta, lam, kw):
    """Values of a large common mean (4 and steps of its bf16 spacing): the recalls come within a percent of them, and the
    differences that rank the pairs are lost in |P|^2 - 2 P.v + |v|^2 (2^-23 |v|^2 = 2e-4 against squared errors of 0.03).
    Selections outside the tie band must be the oracle's."""
    sh = wl.Shape("close", "bf16", 2, 4, 2, d, D, T=0, eta=eta, lam=lam, C=64, seed=0)
    for calls in irregular_calls(eta, lam):
        N = calls[-1][1]
        q, k, v, Wq, Wk = case_inputs(21 + d + D + lam, 2, 4, 2, d, D, N, wscale=0.5 if kw.get("phi_kind") else 1.0)
        v = (4.0 + 2.0 ** -5 * wl.rng(d + lam, 9).integers(-2, 3, v.shape)).astype(np.float32)
        layer, o = None, None
        for a, b in calls:
            print("close", d, D, eta, lam, kw, a, b, flush=True)
            layer, o, _ = P.prefill_parity(sh, q[:, :, a:b], k[:, :, a:b], v[:, :, a:b], Wq, Wk, layer=layer, oracle=o, layer_kw=kw)


@pytest.mark.parametrize("d,D,eta,lam,kw", [(128, 256, 64, 512, {}), (64, 128, 128, 64, {}), (64, 256, 1, 128, {}), (128, 128, 64, 64, dict(score_kind=2))])
def test_step_with_sequences_at_different_stages(d, D, eta, lam, kw):
    """One batch holds an empty sequence, sequences that fill their window or cache at different steps, and one in steady
    state: the same memories, bit for bit, as each sequence stepped by itself; outputs to rounding (their sums over the
    keys may be split differently at another batch size)."""
    n, lens = 4, [0, eta - 1, eta, eta + lam - 2, eta + lam + 70]
    names = FIELDS + (("win_score", "sp_score") if kw else ())
    sh = wl.Shape("stages", "bf16", 1, 4, 2, d, D, T=0, eta=eta, lam=lam, C=64, seed=0)
    q, k, v, Wq, Wk = (case_inputs(70 + d + D, len(lens), 4, 2, d, D, max(lens) + n))
    dq, dk, dv, dWq, dWk = P.to_dev(q, "bf16"), P.to_dev(k, "bf16"), P.to_dev(v, "bf16"), P.w_to_dev(Wq, "bf16"), P.w_to_dev(Wk, "bf16")
    batch = P.make_layer(sh, B=len(lens), **kw)
    alone = []
    for b, T in enumerate(lens):
        lay = P.make_layer(sh, **kw)
        if T:
            lay.prefill(*(x[b:b + 1, :, :T].contiguous() for x in (dq, dk, dv)), dWq, dWk)
        for nm in names:
            getattr(batch, nm)[b].copy_(getattr(lay, nm)[0])
        alone.append(lay)
    for i in range(n):
        tok = [[x[b, :, T + i] for b, T in enumerate(lens)] for x in (dq, dk, dv)]
        out = batch.decode_step(*(torch.stack(x).contiguous() for x in tok), dWq, dWk)
        for b, lay in enumerate(alone):
            o1 = lay.decode_step(*(x[b][None].contiguous() for x in tok), dWq, dWk)
            assert P.row_rel_err(out[b:b + 1].cpu().numpy(), o1.cpu().numpy().astype(np.float64)).max() < 1e-5, (i, b)
            for nm in names:
                assert torch.equal(getattr(batch, nm)[b], getattr(lay, nm)[0]), (i, b, nm)


PIECES = 8   # launches of the state evolution in a pass at most


def shares(layer):
    """What the helpers of the shared evolution did in the last pass of the layer's last call, from the exchange words behind the
    cache slots' features in its workspace: per piece and stream, the helpers that joined and the shares they finished."""
    up = lambda x: (x + 255) // 256 * 256
    ns, rows = layer.B * layer.Hkv, layer.lam + layer.eta
    off = 2 * up(ns * rows * layer.d * 2) + up(ns * layer.lam * 4)
    words = layer.workspace[off:off + ns * (layer.lam + 64) * layer.D * 4].view(torch.int32).view(ns, (layer.lam + 64) * layer.D)
    words = words[:, layer.lam * layer.D:layer.lam * layer.D + PIECES * 96].reshape(ns, PIECES, 96).cpu().numpy()
    return words[:, :, 1].T, words[:, :, 64].T


@pytest.mark.parametrize("B,Hq,d,D,eta,lam,T,first,second", [(8, 32, 128, 256, 128, 256, 2048, True, False), (8, 32, 128, 128, 64, 512, 2048, True, False),
                                                           (2, 32, 128, 256, 64, 1024, 2100, True, True), (4, 32, 128, 256, 512, 1024, 2048, False, False)])
def test_helpers_beside_outputs(B, Hq, d, D, eta, lam, T, first, second):
    """Outputs on the second stream: the first piece, with nothing beside it, has its helpers (if any of its chunks is scored);
    the second piece only where the chain of scored chunks, not the outputs beside it, is what the call waits for."""
    sh = wl.Shape("rule", "bf16", B, Hq, 8, d, D, T=0, eta=eta, lam=lam, C=64, seed=0)
    g = torch.Generator(device=P.DEV).manual_seed(B + lam)
    mk = lambda *shape: torch.randn(shape, generator=g, device=P.DEV).to(torch.bfloat16)
    Wq, Wk = mk(Hq, D // 2, d) / d ** 0.5, mk(8, D // 2, d) / d ** 0.5
    q, k, v = mk(B, Hq, T, d), mk(B, 8, T, d), mk(B, 8, T, d)
    layer = P.make_layer(sh, prefill_overlap=1)
    layer.prefill(q, k, v, Wq, Wk)
    torch.cuda.synchronize()
    joined, done = shares(layer)
    print("helpers", B, Hq, d, D, eta, lam, T, joined.max(1), done.max(1), flush=True)
    assert bool((joined[0] > 0).all()) and bool((done[0] > 0).all()) == first
    assert bool((joined[1] > 0).all()) == bool(joined[1].any()) == second


@pytest.mark.parametrize("B,Hkv,d,D,eta,lam,T,limit,kw", [
    (1, 1, 128, 256, 64, 1024, 1600, None, {}), (1, 3, 64, 256, 128, 512, 1111, None, {}), (4, 8, 128, 128, 64, 512, 2100, None, dict(prefill_overlap=1)),
    (4, 8, 128, 256, 64, 512, 960, None, {}), (1, 2, 64, 128, 64, 768, 1000, 0, {}), (2, 8, 128, 256, 64, 1024, 1537, 40 << 20, dict(phi_kind=1)),
    (2, 8, 128, 256, 64, 1024, 4200, None, dict(prefill_overlap=1)), (4, 4, 128, 256, 128, 256, 4130, None, dict(prefill_overlap=1)), (2, 32, 128, 256, 64, 512, 800, None, {}),
    (1, 8, 128, 128, 128, 128, 900, None, {}), (2, 3, 64, 128, 64, 192, 1010, None, {}), (1, 5, 128, 256, 64, 64, 700, None, {}), (3, 8, 64, 128, 128, 320, 1100, None, {}),
    (1, 2, 128, 256, 192, 128, 1001, None, {}), (4, 8, 128, 256, 64, 192, 1100, None, {}), (2, 8, 64, 256, 64, 192, 900, None, dict(phi_kind=1)), (1, 8, 128, 256, 64, 448, 1300, None, {}), (2, 4, 64, 256, 128, 448, 1400, None, {})])
def test_evolution_shared_among_workgroups(B, Hkv, d, D, eta, lam, T, limit, kw):
    """With outputs and few streams the candidates' scores come from several workgroups per stream; an update-only call
    stays on one. The same instructions on the same operands: the memories agree bit for bit, over several launches and
    workspace passes, a ragged last chunk and a second call that starts with a full cache.  With the outputs beside it the
    evolution runs in pieces of its own, one or several helpers per stream in the first and the second.  The stream's own
    workgroup keeps the batches that it requests ahead (2 with 256 features, 1 with 128) also where there are as many helpers
    as batches: 3, 4, 6, 8 and 16 batches."""
    sh = wl.Shape("shared", "bf16", B, 2 * Hkv, Hkv, d, D, T=0, eta=eta, lam=lam, C=64, seed=0)
    q, k, v, Wq, Wk = case_inputs(90 + d + D + lam, B, 2 * Hkv, Hkv, d, D, T + 130, wscale=0.5 if kw.get("phi_kind") else 1.0)
    dq, dk, dv, dWq, dWk = P.to_dev(q, "bf16"), P.to_dev(k, "bf16"), P.to_dev(v, "bf16"), P.w_to_dev(Wq, "bf16"), P.w_to_dev(Wk, "bf16")
    one, many = P.make_layer(sh, **kw), P.make_layer(sh, **kw)
    for a, b in ((0, T), (T, T + 130)):
        q1, k1, v1 = (x[:, :, a:b].contiguous() for x in (dq, dk, dv))
        print("shared", B, Hkv, d, D, eta, lam, a, b, flush=True)
        out, t_many = many.prefill(q1, k1, v1, dWq, dWk, trace=True, workspace_limit=limit)
        torch.cuda.synchronize()
        joined, done = shares(many)
        print("   helpers", joined.max(1), "shares", done.max(1), flush=True)
        if limit is None:   # (a pass of one chunk may be over before a helper has joined)
            assert bool((joined[0] > 0).all()) and bool((done > 0).any(0).all())
            scored = -(-T // 64) - (eta + lam) // 64 if a == 0 else -(-(b - a) // 64)   # chunks
            assert int(done.sum(0).max()) <= scored * ((lam + 64) // (32 if D == 256 else 64) - (2 if D == 256 else 1))
        if kw.get("prefill_overlap") and a == 0:   # (the second call is too short for pieces)
            assert bool((joined[1] > 0).all()) and bool((done[1] > 0).all())
            apart = P.make_layer(sh)
            assert torch.equal(apart.prefill(q1, k1, v1, dWq, dWk), out)
        _, t_one = one.prefill(None, k1, v1, dWq, dWk, trace=True, workspace_limit=limit)
        torch.cuda.synchronize()
        assert not shares(one)[0].any()
        assert torch.equal(t_many, t_one)
        for nm in FIELDS:
            assert torch.equal(getattr(one, nm), getattr(many, nm)), (a, nm)


def test_filling_chunks_in_a_later_piece():
    """Outputs beside the evolution while the caches still fill in the second piece (24 filling chunks, a first piece of 20): its
    filling chunks share the snapshot that its own launch took.  Outputs and memories as on one stream, bit for bit, then a
    second, ragged call."""
    sh = wl.Shape("later", "bf16", 4, 32, 8, 128, 256, T=0, eta=512, lam=1024, C=64, seed=0)
    g = torch.Generator(device=P.DEV).manual_seed(3)
    mk = lambda *shape: torch.randn(shape, generator=g, device=P.DEV).to(torch.bfloat16)
    Wq, Wk = mk(32, 128, 128) / 128 ** 0.5, mk(8, 128, 128) / 128 ** 0.5
    beside, apart = P.make_layer(sh, prefill_overlap=1), P.make_layer(sh)
    for T in (2048, 77):
        q, k, v = mk(4, 32, T, 128), mk(4, 8, T, 128), mk(4, 8, T, 128)
        out, want = beside.prefill(q, k, v, Wq, Wk), apart.prefill(q, k, v, Wq, Wk)
        torch.cuda.synchronize()
        assert T < 2048 or (int(shares(beside)[0].any(1).sum()) >= 2 and int(shares(apart)[0].any(1).sum()) == 1)   # (pieces)
        assert torch.equal(out, want), T
        for nm in FIELDS:
            assert torch.equal(getattr(beside, nm), getattr(apart, nm)), (T, nm)


def test_shared_evolution_from_two_host_threads():
    """Two host threads, each with a layer, a workspace and a stream of its own, run shared evolutions (48 workgroups each, and the
    outputs beside them) at the same time: each result must be the one that the same call gives alone."""
    import threading
    sh = wl.Shape("threads", "bf16", 1, 16, 8, 128, 256, T=0, eta=64, lam=1024, C=64, seed=0)
    layers, args, want = [], [], []
    for seed in (5, 6):
        q, k, v, Wq, Wk = case_inputs(seed, 1, 16, 8, 128, 256, 2000)
        args.append((P.to_dev(q, "bf16"), P.to_dev(k, "bf16"), P.to_dev(v, "bf16"), P.w_to_dev(Wq, "bf16"), P.w_to_dev(Wk, "bf16")))
        layers.append(P.make_layer(sh))
        want.append((layers[-1].prefill(*args[-1]).clone(), [getattr(layers[-1], nm).clone() for nm in FIELDS]))
        torch.cuda.synchronize()
        assert bool((shares(layers[-1])[1][0] > 0).all())
    outs, errs = [[], []], []

    def run(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(4):
                    layers[i].reset()
                    outs[i].append(layers[i].prefill(*args[i]))
                torch.cuda.current_stream().synchronize()
        except Exception as e:   # surfaced in the main thread
            errs.append(e)

    threads = [threading.Thread(target=run, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errs, errs
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(o, want[i][0]) for o in outs[i])
        for nm, w in zip(FIELDS, want[i][1]):
            assert torch.equal(getattr(layers[i], nm), w), (i, nm)


@pytest.mark.parametrize("d,D,eta,lam,C", [(32, 2, 3, 5, 4), (32, 62, 7, 9, 8), (64, 64, 16, 16, 16), (64, 128, 16, 40, 24), (64, 130, 8, 8, 16),
                                           (256, 64, 5, 31, 16), (64, 48, 33, 17, 40), (128, 80, 0, 3, 7)])
def test_fp32_rows_at_the_edges_of_their_batches(d, D, eta, lam, C):
    """fp32 storage: numbers of projections that divide the workgroup or not, fill a wavefront or exceed it, states smaller and
    larger than a round of fold blocks, candidate counts around the four-row and eight-key batches; against the oracle."""
    sh = wl.Shape("rows", "f32", 1, 2, 1, d, D, T=0, eta=eta, lam=lam, C=C, seed=0)
    g = wl.rng(60 + d + D, 5)
    mk = lambda *shape: g.standard_normal(shape, dtype=np.float32)
    q, k, v = mk(1, 2, 149, d), mk(1, 1, 149, d), mk(1, 1, 149, d)
    Wq, Wk = mk(2, d, D // 2) / np.float32(np.sqrt(d)), mk(1, d, D // 2) / np.float32(np.sqrt(d))
    layer, o = None, None
    for a, b in ((0, 1), (1, 102), (102, 149)):
        layer, o, _ = P.prefill_parity(sh, q[:, :, a:b], k[:, :, a:b], v[:, :, a:b], Wq, Wk, layer=layer, oracle=o)


def test_shared_evolution_replayed_from_a_graph():
    """A captured prefill (emptied memories, 700 + 300 tokens) whose evolution is shared among workgroups: every replay, with
    eager work and a synchronization between, gives the eager call's outputs and memories."""
    sh = wl.Shape("shared_graph", "bf16", 1, 4, 2, 128, 256, T=0, eta=64, lam=512, C=64, seed=0)
    q, k, v, Wq, Wk = case_inputs(17, 1, 4, 2, 128, 256, 1000)
    dq, dk, dv, dWq, dWk = P.to_dev(q, "bf16"), P.to_dev(k, "bf16"), P.to_dev(v, "bf16"), P.w_to_dev(Wq, "bf16"), P.w_to_dev(Wk, "bf16")
    parts = [[x[:, :, a:b].contiguous() for x in (dq, dk, dv)] for a, b in ((0, 700), (700, 1000))]
    eager, lay = P.make_layer(sh), P.make_layer(sh)
    want = [eager.prefill(*p, dWq, dWk) for p in parts]
    outs = [torch.zeros_like(w) for w in want]
    lay.prefill(*parts[0], dWq, dWk, out=outs[0])   # (the workspace is made outside of the capture)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lay.reset()
        for p, o in zip(parts, outs):
            lay.prefill(*p, dWq, dWk, out=o)
    for i in range(4):
        for o in outs:
            o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for o, w in zip(outs, want):
            assert torch.equal(o, w), i
        for nm in FIELDS:
            assert torch.equal(getattr(lay, nm), getattr(eager, nm)), (i, nm)


@pytest.mark.parametrize("B,Hkv,g,d,D,eta,lam,T,kw", [
    (1, 2, 1, 128, 128, 64, 128, 330, {}), (1, 1, 2, 64, 128, 1, 3, 129, {}), (1, 1, 3, 128, 256, 28, 100, 257, {}), (2, 1, 4, 128, 256, 54, 10, 193, {}),
    (1, 1, 4, 64, 256, 65, 127, 385, {}), (1, 1, 6, 128, 128, 200, 0, 300, {}), (1, 1, 8, 64, 256, 7, 64, 200, {}), (1, 1, 4, 128, 128, 64, 64, 64, {}),
    (1, 1, 4, 128, 256, 64, 192, 449, dict(query_hide=1)), (1, 1, 4, 64, 128, 64, 64, 321, dict(query_hide=2)), (1, 2, 2, 128, 128, 40, 72, 331, dict(query_hide=3)),
    (1, 1, 4, 128, 256, 96, 160, 517, dict(phi_kind=1)), (1, 1, 2, 64, 256, 64, 1024, 1300, {}),
    (1, 1, 1, 64, 256, 512, 1024, 333, {}), (2, 1, 4, 128, 256, 128, 512, 577, {}), (1, 2, 2, 128, 128, 320, 192, 449, {}), (1, 1, 2, 64, 128, 192, 0, 130, {}),
    (1, 1, 1, 128, 128, 64, 1024, 70, {}), (1, 1, 6, 64, 128, 64, 256, 200, dict(query_hide=2))])
def test_output_kernel_edges(B, Hkv, g, d, D, eta, lam, T, kw):
    """The chunk-parallel output kernel where its stages are ragged: groups of 1, 2, 4 heads and what is left of others, positions
    that begin inside the first stage, caches and windows that end inside one, a last chunk of few queries, restricted queries,
    stages without a single pair while cache and window fill, a second call that starts inside a chunk.  Against the oracle at
    the bounds of the other shapes."""
    sh = wl.Shape("edges", "bf16", B, g * Hkv, Hkv, d, D, T=0, eta=eta, lam=lam, C=64, seed=0)
    q, k, v, Wq, Wk = case_inputs(300 + d + D + lam + g, B, g * Hkv, Hkv, d, D, T + 70, wscale=0.5 if kw.get("phi_kind") else 1.0)
    print("edges", B, Hkv, g, d, D, eta, lam, T, kw, flush=True)
    layer, o, _ = P.prefill_parity(sh, q[:, :, :T], k[:, :, :T], v[:, :, :T], Wq, Wk, layer_kw=kw)
    P.prefill_parity(sh, q[:, :, T:], k[:, :, T:], v[:, :, T:], Wq, Wk, layer=layer, oracle=o)


@pytest.mark.parametrize("B,Hkv,d,D,eta,lam,kw", [(1, 1, 128, 256, 65, 64, {}), (3, 1, 64, 128, 100, 192, {}), (33, 1, 128, 128, 64, 320, {}), (8, 8, 64, 256, 30, 128, {}),
                                                 (16, 4, 128, 256, 64, 256, dict(phi_kind=1)), (1, 5, 64, 256, 128, 2048, {})])
def test_generation_step_in_groups_of_candidates(B, Hkv, d, D, eta, lam, kw):
    """The step's scores from groups of 32 candidates on several workgroups and its fold in parts of the rows of H^T, at two groups,
    more workgroups than groups, groups that do not divide evenly, 1 to 64 streams, and streams that are still filling: against one
    workgroup per stream (no scratch), every memory equal bit for bit at every step.  Half of the sequences start short of
    a full cache."""
    Hq = 2 * Hkv
    sh = wl.Shape("groups", "bf16", B, Hq, Hkv, d, D, T=0, eta=eta, lam=lam, C=64, seed=0)
    T, nd = eta + lam + 70, 6
    q, k, v, Wq, Wk = case_inputs(500 + d + D + lam, B, Hq, Hkv, d, D, T + nd, wscale=0.5 if kw.get("phi_kind") else 1.0)
    dWq, dWk = P.w_to_dev(Wq, "bf16"), P.w_to_dev(Wk, "bf16")
    print("groups", B, Hkv, d, D, eta, lam, kw, flush=True)
    full, short = P.make_layer(sh, step_scratch=False, **kw), P.make_layer(sh, step_scratch=False, **kw)
    for lay, n in ((full, T), (short, eta + lam - 3)):
        lay.prefill(None, P.to_dev(k[:, :, :n], "bf16"), P.to_dev(v[:, :, :n], "bf16"), None, dWk)
    lays = [P.make_layer(sh, step_scratch=x, **kw) for x in (True, False)]
    assert lays[0].step_scratch is not None
    lays[0].step_scratch.fill_(float("nan"))   # (nothing is read before it is written)
    for lay in lays:
        for nm in FIELDS:
            for b in range(B):
                getattr(lay, nm)[b].copy_(getattr(short if b % 2 else full, nm)[b])
    for i in range(nd):
        sq, sk, sv = (P.to_dev(np.ascontiguousarray(x[:, :, T + i]), "bf16") for x in (q, k, v))
        outs = [lay.decode_step(sq, sk, sv, dWq, dWk) for lay in lays]
        torch.cuda.synchronize()
        assert torch.allclose(outs[0], outs[1], rtol=1e-5, atol=2e-6), i
        for nm in FIELDS:
            assert torch.equal(getattr(lays[0], nm), getattr(lays[1], nm)), (i, nm)


@pytest.mark.parametrize("B,Hkv,d,D,eta,lam,kw", [(1, 2, 128, 256, 65, 256, {}), (3, 1, 64, 128, 100, 192, {}), (8, 8, 128, 128, 30, 256, {}), (4, 4, 64, 256, 128, 320, {}),
                                                 (2, 4, 128, 256, 64, 512, dict(phi_kind=1)), (16, 4, 128, 128, 128, 64, {}), (9, 8, 128, 256, 64, 512, {}), (8, 8, 64, 128, 64, 512, {}), (4, 8, 64, 256, 64, 1024, {})])
def test_generation_step_ranks_ties_alike_with_the_scratch(B, Hkv, d, D, eta, lam, kw):
    """Which pair leaves does not depend on whether the step has the scratch, also where the scores are equal up to their last
    bits: every value is a permutation of one vector, H and s hold one number each, so that the recalls of all pairs are the same
    number and the scores differ by the rounding of their sums alone.  Every memory equal bit for bit at every step."""
    Hq = 2 * Hkv
    sh = wl.Shape("ties", "bf16", B, Hq, Hkv, d, D, T=0, eta=eta, lam=lam, C=64, seed=0)
    T, nd = eta + lam + 70, 12
    q, k, v, Wq, Wk = case_inputs(700 + d + D + lam, B, Hq, Hkv, d, D, T + nd, wscale=0.5 if kw.get("phi_kind") else 1.0)
    v = wl.rng(d + lam, 11).permuted(np.broadcast_to(v[:1, :1, :1], v.shape), axis=-1)
    dWq, dWk = P.w_to_dev(Wq, "bf16"), P.w_to_dev(Wk, "bf16")
    print("ties", B, Hkv, d, D, eta, lam, kw, flush=True)
    lays = [P.make_layer(sh, step_scratch=x, **kw) for x in (True, False)]
    lays[1].prefill(None, P.to_dev(np.ascontiguousarray(k[:, :, :T]), "bf16"), P.to_dev(np.ascontiguousarray(v[:, :, :T]), "bf16"), None, dWk)
    for nm in FIELDS:
        getattr(lays[0], nm).copy_(getattr(lays[1], nm))
    for i in range(nd):
        sq, sk, sv = (P.to_dev(np.ascontiguousarray(x[:, :, T + i]), "bf16") for x in (q, k, v))
        for lay in lays:
            lay.H.fill_(0.37)
            lay.s.fill_(0.53)
            lay.decode_step(sq, sk, sv, dWq, dWk)
        torch.cuda.synchronize()
        for nm in FIELDS:
            assert torch.equal(getattr(lays[0], nm), getattr(lays[1], nm)), (i, nm)


def test_outputs_of_more_heads_than_a_grid_has_threads():
    """65 535 sequences of 513 query heads on one memory each: with one workgroup per head and chunk in the grid's first dimension
    it would pass 2^32 threads, more than a launch takes.  The first, a middle and the last sequence against layers of their own."""
    from paper_2505_23666_amd import binding as lb
    B, Hq, d, D = 65535, 513, 64, 128
    torch.cuda.empty_cache()
    g = torch.Generator(device=P.DEV).manual_seed(8)
    mk = lambda *shape: torch.randn(shape, generator=g, device=P.DEV, dtype=torch.bfloat16)
    q, k, v, Wq, Wk = mk(B, Hq, 1, d), mk(B, 1, 1, d), mk(B, 1, 1, d), mk(Hq, D // 2, d) / 8, mk(1, D // 2, d) / 8
    lay = lb.LolaLayer(B, Hq, 1, d, D, 0, 0, 64, out_dtype="bf16")
    assert lay.lola_path[0] == "mixed"
    H, s = torch.randn((d, D), generator=g, device=P.DEV), torch.rand((D,), generator=g, device=P.DEV)
    lay.H.copy_(H), lay.s.copy_(s)
    out = lay.prefill(q, k, v, Wq, Wk)
    torch.cuda.synchronize()
    for b in (0, 40000, B - 1):
        one = lb.LolaLayer(1, Hq, 1, d, D, 0, 0, 64, out_dtype="bf16")
        one.H.copy_(H), one.s.copy_(s)
        want = one.prefill(*(x[b:b + 1].contiguous() for x in (q, k, v)), Wq, Wk)
        assert float(want.float().std()) > 0 and torch.equal(out[b], want[0]), b
    del q, out, lay
    torch.cuda.empty_cache()
