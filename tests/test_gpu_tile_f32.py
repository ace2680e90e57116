"""GPU tests of the fp32 score tiles (rows beyond the short-row kernel, d a multiple of 16):
against the fp64 oracle around the 128-query, 32-query and 64-key tile edges, the 16-feature
steps and the diagonal, and the same bits whatever the chunk."""
import pytest
import torch

import paper_2106_06899_amd as tk
from paper_2106_06899_amd import workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu

# (H, Lq, Lk, d, k, chunk, causal); d = 8 keeps the scalar kernel
CASES = [
    (1, 1, 1025, 16, 5, 1, False), (2, 33, 1087, 48, 33, 32, False), (1, 129, 1089, 96, 100, 129, False),
    (2, 1100, 1100, 64, 40, 127, True), (1, 70, 1028, 272, 12, 64, False), (3, 31, 63, 16, 7, 5, False),
    (1, 300, 130, 256, 20, 128, True), (1, 40, 1200, 8, 9, 40, False),
    # causal heads share the chip eight at a time, the rest tile by tile
    (9, 230, 1100, 32, 12, 64, True), (3, 1300, 1300, 16, 30, 500, True), (16, 150, 1030, 16, 8, 150, True),
]


@pytest.mark.parametrize("case", CASES)
def test_fp32_score_tiles(case):
    H, Lq, Lk, d, k, chunk, causal = case
    w = wl.WORKLOADS["c1"].scaled(H=H, Lq=Lq, Lk=Lk, d=d, k=k, chunk=chunk, causal=causal)
    print("[case]", w, flush=True)
    x = wl.make_inputs(w)
    out, idx, _ = parity.run_attn(w, x)
    parity.check_attn(w, x, out, idx, rows=parity.sample_attn_rows(w, min(300, H * Lq), seed=6))
    other = parity.run_attn(w.scaled(chunk=50), x, debug=False)
    assert torch.equal(other, out)


def test_fp32_scores_of_many_chunks():
    """Chunks of one row in such numbers that one launch cannot hold their tiles: the same scores, bit
    for bit, as in chunks of 1024."""
    gen = torch.Generator(device="cuda").manual_seed(2)
    q, k = torch.randn(1, 1, 60000, 48, generator=gen, device="cuda"), torch.randn(1, 1, 20000, 48, generator=gen, device="cuda")
    ref = tk.attn(q, k, k, 8, 1024, cache=True)
    for a, b in zip(ref, tk.attn(q, k, k, 8, 1, cache=True)):
        assert torch.equal(a, b)
