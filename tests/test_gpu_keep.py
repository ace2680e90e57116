"""GPU tests of the select that keeps its lists' order (the filtered path's scan, d = 128, k >
64): against the fp64 oracle at the edges of its sizes, under the causal mask (rows with
fewer keys than k) and not, with the cache outputs sorted and the same output bits without
them; ties at the k-th score."""
import numpy as np
import pytest
import torch

import paper_2106_06899_amd as tk
from paper_2106_06899_amd import workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu


def _check(w, x):
    assert tk.attn_path(w.B, w.H, w.Lq, w.Lk, w.d, w.k, w.chunk, w.causal) == 4
    out, idx, sc = parity.run_attn(w, x)
    parity.check_attn(w, x, out, idx, rows=parity.sample_attn_rows(w, 80, seed=2))
    s, g = sc.cpu().numpy().reshape(-1, w.k), idx.cpu().numpy().reshape(-1, w.k)
    keep = g[:, 1:] >= 0
    assert np.all((s[:, 1:] < s[:, :-1])[keep] | ((s[:, 1:] == s[:, :-1]) & (g[:, 1:] > g[:, :-1]))[keep])
    assert torch.equal(parity.run_attn(w, x, debug=False), out)


@pytest.mark.parametrize("k", [65, 128, 129, 256, 257, 512])
@pytest.mark.parametrize("causal", [False, True])
def test_select_in_list_order(k, causal):
    w = wl.WORKLOADS["c4"].scaled(B=1, H=2, Lq=1400, Lk=2500, k=k, causal=causal, chunk=500)
    print("[case]", w, flush=True)
    _check(w, wl.make_inputs(w))


def test_select_in_list_order_ties():
    """Every key four times over: the k-th score is tied in most rows."""
    w = wl.WORKLOADS["c4"].scaled(B=1, H=1, Lq=300, Lk=3000, k=90, causal=False, chunk=500)
    x = wl.make_inputs(w)
    kv = x["K"].values[0, 0]
    kv[:] = kv[np.arange(w.Lk) // 4 * 4]
    x["K"] = wl._store(kv[None, None], w.dtype)
    print("[case] ties", w, flush=True)
    _check(w, x)
