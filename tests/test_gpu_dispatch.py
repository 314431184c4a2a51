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
