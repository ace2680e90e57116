"""GPU tests of the short-row kernel (rows of at most 1024 keys, k <= 256, d = 32, 64, 96
or 128): against the fp64 oracle at the edges of its key groups, row tiles and outputs,
ties at the k-th score, and value rows that are not finite."""
import numpy as np
import pytest
import torch

import paper_2106_06899_amd as tk
from paper_2106_06899_amd import workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu

# (B, H, Lq, Lk, d, k, causal): key counts around the 64-key waves and the 256- and
# 512-key kernel sizes; row counts around the 16- and 32-row tiles; 512 heads fill enough
# workgroups for 32-row tiles; k around the sizes of the cache outputs' sort
CASES = [
    (1, 1, 1, 1, 32, 1, False), (1, 2, 17, 63, 64, 64 - 1, False), (1, 1, 33, 65, 96, 64, False),
    (1, 1, 15, 255, 128, 65, True), (2, 1, 16, 256, 64, 128, False), (1, 1, 40, 257, 32, 129, False),
    (1, 2, 530, 511, 64, 20, True), (1, 1, 31, 513, 96, 256, False), (1, 1, 20, 1000, 128, 200, False),
    (1, 1, 1100, 1024, 64, 100, True), (16, 32, 33, 130, 64, 40, False), (32, 16, 31, 520, 128, 128, False),
    (16, 32, 20, 300, 96, 3, True), (16, 32, 5, 1024, 32, 200, False),
    # the 32-row kernels of d = 128 that keep some registers in scratch memory
    (16, 32, 33, 250, 128, 60, False), (16, 32, 20, 500, 128, 100, True),
    # 16 rows a workgroup with the cache outputs (their sort scratch), 32 without
    (16, 32, 40, 400, 64, 200, True),
    # as many kept keys as the sorts of the cache outputs hold, and one more
    (1, 2, 50, 300, 64, 8, True), (1, 2, 50, 300, 64, 9, False), (1, 2, 50, 600, 32, 32, True), (1, 2, 50, 200, 64, 33, True),
]


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("case", CASES)
def test_short_rows(case, dtype):
    B, H, Lq, Lk, d, k, causal = case
    w = wl.WORKLOADS["c2"].scaled(B=B, H=H, Lq=Lq, Lk=Lk, d=d, k=k, causal=causal, dtype=dtype, chunk=7)
    print("[case]", w, flush=True)
    assert tk.attn_workspace_bytes(B, H, Lq, Lk, d, k, 7, causal, tk.TOPK_BF16 if dtype == wl.BF16 else tk.TOPK_F32) == 256
    x = wl.make_inputs(w)
    out, idx, sc = parity.run_attn(w, x)
    rows = parity.sample_attn_rows(w, min(400, B * H * Lq), seed=5)
    parity.check_attn(w, x, out, idx, rows=rows)
    # every row: k_eff distinct valid keys, and the same bits without the cache outputs
    g = idx.cpu().numpy().reshape(B * H, Lq, k)
    k_eff = np.minimum(k, np.arange(Lq) + 1) if causal else np.full(Lq, k)
    assert np.array_equal((g >= 0).sum(-1), np.broadcast_to(np.minimum(k_eff, Lk), (B * H, Lq)))
    s = sc.cpu().numpy().reshape(B * H, Lq, k)
    assert np.array_equal(np.isneginf(s), g < 0)
    assert torch.equal(parity.run_attn(w, x, debug=False), out)


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("Lk,k", [(200, 64), (700, 100), (1024, 256)])
def test_short_rows_ties(Lk, k, dtype):
    """Scores that take four values only (keys repeated): the k-th is always tied, and the
    lowest indices among the tied keys are kept."""
    w = wl.WORKLOADS["c2"].scaled(B=1, H=1, Lq=40, Lk=Lk, k=k, dtype=dtype)
    x = wl.make_inputs(w)
    kv = x["K"].values[0, 0]
    kv[:] = kv[np.arange(Lk) % 4]
    x["K"] = wl._store(kv[None, None], dtype)
    print("[case] ties", w, flush=True)
    out, idx, _ = parity.run_attn(w, x)
    s = x["Q"].values[0, 0].astype(np.float64) @ kv[:4].astype(np.float64).T
    g = idx.cpu().numpy()[0, 0]
    for i in range(w.Lq):
        order = sorted(range(Lk), key=lambda j: (-s[i, j % 4], j))[:k]
        assert g[i].tolist() == order
    parity.check_attn(w, x, out, idx)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_short_rows_value_rows_not_finite(dtype):
    """Unselected value rows that are infinite or NaN do not reach the output; a selected
    one does, in its column only."""
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn(1, 2, n, 64, generator=gen, device="cuda").to(dtype) for n in (50, 300, 300))
    ref, idx, _ = tk.attn(q, k, v, 8, cache=True)
    used = torch.zeros(2, 300, dtype=torch.bool, device="cuda")
    for h in range(2):
        used[h, idx[0, h].flatten().long()] = True
    free = (~used[0]).nonzero().flatten()
    assert free.numel() >= 2
    v2 = v.clone()
    v2[0, 0, free[0]] = float("inf")
    v2[0, 0, free[1]] = float("nan")
    got = tk.attn(q, k, v2, 8)
    tol = 2e-2 if dtype == torch.bfloat16 else 1e-5
    assert torch.isfinite(got).all()
    assert ((got - ref).abs().max(-1).values <= tol * ref.abs().max(-1).values).all()
    v3 = v2.clone()
    v3[0, 1, idx[0, 1, 0, 0].long(), 5] = float("inf")
    got = tk.attn(q, k, v3, 8)
    bad = ~torch.isfinite(got)
    rows = (idx[0, 1] == idx[0, 1, 0, 0]).any(-1)
    want = torch.zeros_like(bad)
    want[0, 1, :, 5] = rows
    assert torch.equal(bad, want)


@pytest.mark.parametrize("d", [32, 64, 96, 128])
@pytest.mark.parametrize("dff,N", [(200, 40), (400, 40), (1000, 40), (130, 17000)])
def test_short_rows_keep_32_bits(dff, N, d):
    """Weights (ReLU scores) of 18 significant bits that cancel to their last bits: exact in 32 bits,
    lost in 16."""
    gen = torch.Generator(device="cuda").manual_seed(7)
    row = lambda *v: torch.cat([torch.tensor(v, device="cuda"), torch.zeros(d - len(v), device="cuda")])
    x, w1, w2 = torch.zeros(N, d, device="cuda"), torch.zeros(dff, d, device="cuda"), torch.zeros(dff, d, device="cuda")
    x[:] = row(256.0, 1, 1)
    w1[3], w1[dff - 2] = row(512.0, 256, 1), row(512.0, 0, 255)  # scores 2^17 + 257 and 2^17 + 255
    w2[3] = torch.randint(-100, 100, (d,), generator=gen, device="cuda")
    w2[dff - 2] = -w2[3]
    out = tk.ffn(*(t.bfloat16() for t in (x, w1, w2)), 2)
    assert torch.equal(out.float(), (2 * w2[3]).expand(N, -1))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("Lk,k", [(100, 8), (300, 8), (1000, 8), (200, 200)])
def test_short_rows_tiny_weights(Lk, k, dtype):
    """A weight below the smallest normal number (2^-130) against a value of 2^120."""
    q, kk, v = (torch.zeros(1, 1, n, 64, device="cuda") for n in (40, Lk, Lk))
    q[..., 0] = 1
    kk[0, 0, :, 0] = -1e4
    kk[0, 0, 0, 0], kk[0, 0, 1, 0] = 0, -90.0 * 8
    v[0, 0, 1] = 2.0 ** 120
    out = tk.attn(q.to(dtype), kk.to(dtype), v.to(dtype), k, 0, False, 0.125).double()
    want = np.exp(-90.0) * 2.0 ** 120
    # the weight has 19 bits; its exponent, 130, an error of 2^-17 at most
    tol = 2.0 ** -16 + (2.0 ** -8 if dtype == torch.bfloat16 else 0)
    assert bool(((out - want).abs() <= tol * want).all()), out.flatten()[0]


def test_short_rows_beyond_one_launch():
    """More workgroups than one launch can hold (2^32 threads): 2^24 and some heads of one key."""
    B, H = 4096, 4104
    gen = torch.Generator(device="cuda").manual_seed(3)
    q = torch.ones(B, H, 1, 32, device="cuda", dtype=torch.bfloat16)
    v = torch.empty_like(q)
    for b in range(0, B, 512):
        v[b:b + 512] = torch.randn(512, H, 1, 32, generator=gen, device="cuda")
    assert torch.equal(tk.attn(q, q, v, 1), v)


# calls of short rows that run as chunk tiles or with the few-query kernels
LEFT = [(1, 1, 300, 1024, 128, 8, False, torch.float32), (1, 16, 1030, 600, 128, 20, True, torch.bfloat16),
        (1, 900, 2, 1000, 64, 40, False, torch.bfloat16)]


@pytest.mark.parametrize("case", LEFT)
def test_short_rows_in_a_workspace_too_small_for_the_general_paths(case):
    """The short-row kernel, which needs none, runs them there."""
    B, H, Lq, Lk, d, k, causal, dtype = case
    print("[case]", case, flush=True)
    dt = tk.TOPK_BF16 if dtype == torch.bfloat16 else tk.TOPK_F32
    assert tk.attn_workspace_bytes(B, H, Lq, Lk, d, k, 0, causal, dt) > 256
    gen = torch.Generator(device="cuda").manual_seed(11)
    q, kk, v = (torch.randn(B, H, n, d, generator=gen, device="cuda").to(dtype) for n in (Lq, Lk, Lk))
    ref, got = tk.attn(q, kk, v, k, 0, causal, 0.1), torch.empty_like(q)
    ws = torch.empty(4096, dtype=torch.uint8, device="cuda")
    tk._raise(tk.lib().topk_set_workspace(ws.data_ptr(), 4096))
    try:
        tk._raise(tk.lib().topk_attn(q.data_ptr(), kk.data_ptr(), v.data_ptr(), got.data_ptr(), B, H, Lq, Lk, d, k, 0, int(causal), 0.1, dt,
                                     torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
    finally:
        tk.lib().topk_set_workspace(None, 0)
    # sums in another order; in bf16 a result on the other side of a rounding (2^-8)
    tol = 2.0 ** -7 if dtype == torch.bfloat16 else 1e-5
    assert bool(((got.float() - ref.float()).abs().amax(-1) <= tol * ref.float().abs().amax(-1)).all())


def test_short_rows_as_chunk_tiles_in_the_fixed_scratch():
    """Whatever the chunk: the tiles of at most 1024 rows at a time."""
    gen = torch.Generator(device="cuda").manual_seed(12)
    q = torch.randn(1, 1, 70000, 128, generator=gen, device="cuda").bfloat16()
    kk, v = (torch.randn(1, 1, 1000, 128, generator=gen, device="cuda").bfloat16() for _ in range(2))
    assert tk.attn_workspace_bytes(1, 1, 70000, 1000, 128, 8, 70000, True) > 256
    ref = tk.attn(q, kk, v, 8, 512, True, 0.1)
    assert torch.equal(tk.attn(q, kk, v, 8, 70000, True, 0.1), ref)
    got = torch.empty_like(q)
    tk._raise(tk.lib().topk_attn_noalloc(q.data_ptr(), kk.data_ptr(), v.data_ptr(), got.data_ptr(), 1, 1, 70000, 1000, 128, 8, 70000, 1, 0.1,
                                         tk.TOPK_BF16, torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert torch.equal(got, ref)
