"""GPU tests of the backward pass by cells (64 x 64 blocks of selected pairs expanded into
matrix products): against the fp64 oracle at the edges of its strips, cells and tiles and
with split products; equal to the gathers by lists within rounding; keys listed twice in a
row, padding, and rows that are not finite."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2106_06899_amd as tk
from oracle import topk_backward as bo
from paper_2106_06899_amd import workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu


def _lists(fn):
    tk.set_backward_lists(tk.TOPK_LISTS_BUCKET)
    try:
        return fn()
    finally:
        tk.set_backward_lists(tk.TOPK_LISTS_AUTO)


def _attn_by_cells(B, H, Lq, Lk, d, k):
    """Whether such a backward pass runs by cells: its workspace is not the lists'."""
    f = lambda: tk.lib().topk_attn_backward_workspace_bytes(B, H, Lq, Lk, d, k, tk.TOPK_BF16)
    return f() != _lists(f)


def _ffn_by_cells(N, dm, dff, k):
    f = lambda: tk.lib().topk_ffn_backward_workspace_bytes(N, dm, dff, k, tk.TOPK_BF16)
    return f() != _lists(f)


def _close(a, b):
    """Two bf16 results of the same sums in different orders: neighbouring bf16 numbers at
    most, which lie up to 2^-7 of their size apart; held to each row's largest entry."""
    a, b = a.float(), b.float()
    tol = 2.0 ** -7 * b.abs().amax(-1, keepdim=True) + 1e-6 * b.abs().max()
    assert bool(((a - b).abs() <= tol).all()), float(((a - b).abs() / tol.clamp_min(1e-30)).max())


# rows around the 64-row strips and 128-row tiles, units around the 64-key cells (4096 units
# of few rows split the products); column tiles of 256 that d fills, half fills and repeats; the
# most units a strip's bitmap holds
FFN_CASES = [(1, 512, 64, 64), (63, 768, 300, 64), (65, 288, 129, 129), (130, 1024, 513, 70), (300, 512, 4096, 171),
             (257, 256, 2000, 512), (100, 512, 16384, 410), (70, 512, 16377, 410)]


@pytest.mark.parametrize("case", FFN_CASES)
def test_ffn_cells(case):
    N, dm, dff, k = case
    assert _ffn_by_cells(*case)
    w = wl.WORKLOADS["c5"].scaled(N=N, d_model=dm, d_ff=dff, k=k, chunk=64)
    print("[case]", w, flush=True)
    x = wl.make_inputs(w)
    a, b1, b2 = (parity.to_dev(x[n]) for n in ("X", "W1", "W2"))
    _, idx, dots = tk.ffn(a, b1, b2, k, w.chunk, cache=True)
    g = parity.grad_out((N, dm), w.dtype, 31)
    got = tk.ffn_backward(a, b1, b2, idx, dots, parity.to_dev(g))
    ref, mag = bo.oracle_ffn_backward(x["X"].values, x["W1"].values, x["W2"].values, idx.cpu().numpy(), g.values,
                                      chunk=64, magnitudes=True)
    for n, p, r, m in zip(("d_X", "d_W1", "d_W2"), got, ref, mag):
        parity.check_grad_rows(n, p, r, m, w.dtype)


# enough heads for the rules of d = 128 (128 tiles) and d = 64 (256 tiles)
ATTN_CASES = [(8, 16, 70, 90, 128, 20, False), (8, 16, 70, 70, 128, 20, True), (16, 16, 65, 65, 64, 9, True),
              (4, 8, 500, 130, 128, 100, False), (2, 128, 33, 40, 160, 40, False)]


@pytest.mark.parametrize("case", ATTN_CASES)
def test_attention_cells(case):
    B, H, Lq, Lk, d, k, causal = case
    assert _attn_by_cells(B, H, Lq, Lk, d, k)
    w = wl.WORKLOADS["c4"].scaled(B=B, H=H, Lq=Lq, Lk=Lk, d=d, k=k, causal=causal, scale=float(np.float32(d ** -0.5)))
    print("[case]", w, flush=True)
    x = wl.make_inputs(w)
    q, kk, v = (parity.to_dev(x[n]) for n in ("Q", "K", "V"))
    _, idx, dots = tk.attn(q, kk, v, k, 64, causal, w.scale, cache=True)
    g = parity.grad_out((B, H, Lq, d), w.dtype, 32)
    gd = parity.to_dev(g)
    got = tk.attn_backward(q, kk, v, idx, dots, gd, w.scale)
    again = tk.attn_backward(q, kk, v, idx, dots, gd, w.scale)
    for p, r in zip(got, again):
        assert torch.equal(p, r)
    hs = [0, H // 2, H - 1]  # three heads of the last batch against the oracle
    sub = [t.values[-1:, hs] for t in (x["Q"], x["K"], x["V"])]
    ref, mag = bo.oracle_attn_backward(*sub, idx[-1:, hs].cpu().numpy(), g.values[-1:, hs], w.scale, chunk=64, magnitudes=True)
    for n, p, r, m in zip(("d_Q", "d_K", "d_V"), got, ref, mag):
        parity.check_grad_rows(n, p[-1:, hs], r, m, w.dtype)
    for p, r in zip(got, _lists(lambda: tk.attn_backward(q, kk, v, idx, dots, gd, w.scale))):
        _close(p, r)


@pytest.mark.parametrize("causal", [False, True])
def test_attention_cells_long_products(causal):
    """12 heads of 4200: products of 66 cells in one part (the ranges are read 64 cells at a time), more
    pairs a strip (17920) than the softmax's pass holds in registers. One head against the oracle
    at sampled rows and keys."""
    H, L, d, k = 12, 4200, 128, 280
    assert _attn_by_cells(1, H, L, L, d, k)
    w = wl.WORKLOADS["c4"].scaled(B=1, H=H, Lq=L, Lk=L, d=d, k=k, causal=causal, scale=float(np.float32(d ** -0.5)))
    print("[case]", w, flush=True)
    x = wl.make_inputs(w)
    q, kk, v = (parity.to_dev(x[n]) for n in ("Q", "K", "V"))
    _, idx, dots = tk.attn(q, kk, v, k, 0, causal, w.scale, cache=True)
    g = parity.grad_out((1, H, L, d), w.dtype, 33)
    gd = parity.to_dev(g)
    got = tk.attn_backward(q, kk, v, idx, dots, gd, w.scale)
    for p, r in zip(got, tk.attn_backward(q, kk, v, idx, dots, gd, w.scale)):
        assert torch.equal(p, r)
    for p, r in zip(got, _lists(lambda: tk.attn_backward(q, kk, v, idx, dots, gd, w.scale))):
        _close(p, r)
    rows = np.array([0, 1, 63, 64, 300, 4095, 4096, 4150, L - 1])
    keys = np.array([0, 5, 63, 64, 1000, 4095, 4096, 4100])
    hd = H - 1
    ref, mag = bo.sampled_backward(*(x[n].values[0, hd] for n in ("Q", "K", "V")), idx[0, hd].cpu().numpy(), g.values[0, hd],
                                   rows, keys, "softmax", w.scale, magnitudes=True)
    for n, p, at, r, m in zip(("d_Q", "d_K", "d_V"), got, (rows, keys, keys), ref, mag):
        parity.check_grad_rows(n, p[0, hd][torch.from_numpy(at).cuda()], r, m, w.dtype)


def test_cells_keys_listed_twice_and_padding():
    """A caller's own index lists: keys repeated in a row add up, entries outside the keys
    are padding; as by lists."""
    gen = torch.Generator(device="cuda").manual_seed(4)
    x, g = (torch.randn(200, 256, generator=gen, device="cuda").bfloat16() for _ in range(2))
    w1, w2 = (torch.randn(500, 256, generator=gen, device="cuda").bfloat16() for _ in range(2))
    assert _ffn_by_cells(200, 256, 500, 128)
    idx = torch.randint(-3, 520, (200, 128), generator=gen, device="cuda", dtype=torch.int32)
    idx[:64] = torch.stack([torch.randperm(500, generator=gen, device="cuda")[:128] for _ in range(64)]).int()  # a strip without repeats
    dots = torch.randn(200, 128, generator=gen, device="cuda")
    got = tk.ffn_backward(x, w1, w2, idx, dots, g)
    for p, r in zip(got, _lists(lambda: tk.ffn_backward(x, w1, w2, idx, dots, g))):
        _close(p, r)


@pytest.mark.parametrize("N,dff", [(400, 1000), (140, 4000)])  # whole products, split products
def test_cells_rows_not_finite(N, dff):
    """An infinite row of d_out reaches its own d_X row and the units its token kept, nothing
    else; the rest is what it is without it."""
    gen = torch.Generator(device="cuda").manual_seed(5)
    x, g = (torch.randn(N, 256, generator=gen, device="cuda").bfloat16() for _ in range(2))
    w1, w2 = (torch.randn(dff, 256, generator=gen, device="cuda").bfloat16() for _ in range(2))
    k = 128 if dff == 1000 else 256
    assert _ffn_by_cells(N, 256, dff, k)
    _, idx, dots = tk.ffn(x, w1, w2, k, cache=True)
    ref = _lists(lambda: tk.ffn_backward(x, w1, w2, idx, dots, g))
    bad = g.clone()
    bad[70] = float("inf")
    got = tk.ffn_backward(x, w1, w2, idx, dots, bad)
    lst = _lists(lambda: tk.ffn_backward(x, w1, w2, idx, dots, bad))
    for p, q, r in zip(got, lst, ref):
        fin = torch.isfinite(q).all(-1)
        assert torch.equal(torch.isfinite(p).all(-1), fin)
        assert 0 < int((~fin).sum()) < p.shape[0]
        _close(p[fin], r[fin])


def test_cells_need_more_workspace_than_lists():
    """A registered workspace that holds the lists but not the cells is still enough."""
    L = tk.lib()
    gen = torch.Generator(device="cuda").manual_seed(6)
    x, g = (torch.randn(512, 1024, generator=gen, device="cuda").bfloat16() for _ in range(2))
    w1, w2 = (torch.randn(4096, 1024, generator=gen, device="cuda").bfloat16() for _ in range(2))
    _, idx, dots = tk.ffn(x, w1, w2, 128, cache=True)
    cells = L.topk_ffn_backward_workspace_bytes(512, 1024, 4096, 128, tk.TOPK_BF16)
    lists = _lists(lambda: L.topk_ffn_backward_workspace_bytes(512, 1024, 4096, 128, tk.TOPK_BF16))
    assert cells > lists  # split products
    want = _lists(lambda: tk.ffn_backward(x, w1, w2, idx, dots, g))
    out = [torch.empty_like(t) for t in (x, w1, w2)]
    ws = torch.empty(lists, dtype=torch.uint8, device="cuda")
    tk._raise(L.topk_set_workspace(ctypes.c_void_p(ws.data_ptr()), lists))
    try:
        tk._raise(L.topk_ffn_backward(x.data_ptr(), w1.data_ptr(), w2.data_ptr(), idx.data_ptr(), dots.data_ptr(), g.data_ptr(),
                                      out[0].data_ptr(), out[1].data_ptr(), out[2].data_ptr(), 512, 1024, 4096, 128, tk.TOPK_BF16,
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    finally:
        L.topk_set_workspace(None, 0)
    torch.cuda.synchronize()
    for p, r in zip(out, want):
        assert torch.equal(p, r)


def test_cells_where_the_lists_do_not_fit():
    """A registered workspace that holds the cells of a call that the lists finish sooner, but not the
    lists: many pairs in unsplit products."""
    L = tk.lib()
    B, H, n, d, k = 1, 24, 2048, 64, 512
    assert not _attn_by_cells(B, H, n, n, d, k)
    lists = L.topk_attn_backward_workspace_bytes(B, H, n, n, d, k, tk.TOPK_BF16)
    gen = torch.Generator(device="cuda").manual_seed(13)
    q, kk, v, g = (torch.randn(B, H, n, d, generator=gen, device="cuda").bfloat16() for _ in range(4))
    _, idx, dots = tk.attn(q, kk, v, k, cache=True)
    want = tk.attn_backward(q, kk, v, idx, dots, g)
    out = [torch.empty_like(q) for _ in range(3)]
    size = lists * 3 // 4 // 256 * 256
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    tk._raise(L.topk_set_workspace(ctypes.c_void_p(ws.data_ptr()), size))
    try:
        tk._raise(L.topk_attn_backward(q.data_ptr(), kk.data_ptr(), v.data_ptr(), idx.data_ptr(), dots.data_ptr(), g.data_ptr(), out[0].data_ptr(),
                                       out[1].data_ptr(), out[2].data_ptr(), B, H, n, n, d, k, d ** -0.5, tk.TOPK_BF16,
                                       ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    finally:
        L.topk_set_workspace(None, 0)
    torch.cuda.synchronize()
    for p, r in zip(out, want):
        _close(p, r)


@pytest.mark.parametrize("dm", [256, 288, 1024])
def test_cells_keep_32_bits(dm):
    """Weights and score gradients of 18 significant bits that cancel to their last bits: exact in 32
    bits (products of 18-bit integers and powers of two, sums that stay below 2^24), lost in 16."""
    N, dff, k = 300, 700, 128
    assert _ffn_by_cells(N, dm, dff, k)
    gen = torch.Generator(device="cuda").manual_seed(7)
    pow2 = lambda *s: (torch.randint(0, 2, s, generator=gen, device="cuda") * 2 - 1) * 2.0 ** torch.randint(-1, 2, s, generator=gen, device="cuda")
    big, near = 2.0 ** 17 + 257, 2.0 ** 17 + 255
    row = lambda *v: torch.cat([torch.tensor(v, device="cuda"), torch.zeros(dm - len(v), device="cuda")])
    x, w1, w2, g = pow2(N, dm), pow2(dff, dm), pow2(dff, dm), pow2(N, dm)
    idx = torch.full((N, k), -1, dtype=torch.int32, device="cuda")
    dots = torch.ones(N, k, device="cuda")
    # units 0 .. 29, kept by tokens 0 and 100: their score gradients are `big` and `-near`
    x[100] = x[0]
    w2[:30], g[0], g[100] = row(512, 256, 1), row(256, 1, 1), row(-256, 0, -255)
    idx[[0, 100], :30] = torch.arange(30, dtype=torch.int32, device="cuda")
    # units 600 .. 629, kept by tokens 5 and 290 with weights `big` and `near`
    g[290] = -g[5]
    idx[[5, 290], :30] = torch.arange(600, 630, dtype=torch.int32, device="cuda")
    dots[5], dots[290] = big, near
    # token 70 keeps units 300 and 500: score gradients `big` and `-near`
    w1[500] = w1[300]
    w2[300], w2[500], g[70] = row(512, 256, 1), row(-512, 0, -255), row(256, 1, 1)
    idx[70, 3], idx[70, 9] = 300, 500
    dx, dw1, dw2 = tk.ffn_backward(*(t.bfloat16() for t in (x, w1, w2)), idx, dots, g.bfloat16())
    assert torch.equal(dw1[:30].float(), (2 * x[0]).expand(30, -1))
    assert torch.equal(dw2[600:630].float(), (2 * g[5]).expand(30, -1))
    assert torch.equal(dx[70].float(), 2 * w1[300])
    # weights as small as floats get (multiples of 2^-149)
    g[5] *= 2.0 ** 100
    g[290] = -g[5]
    dots[5], dots[290] = dots[5] * 2.0 ** -100 * 2.0 ** -49, dots[290] * 2.0 ** -100 * 2.0 ** -49
    dw2 = tk.ffn_backward(*(t.bfloat16() for t in (x, w1, w2)), idx, dots, g.bfloat16())[2]
    assert torch.equal(dw2[600:630].double(), (2.0 ** -148 * g[5].double()).expand(30, -1))


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_cells_closed_gate_at_a_key_that_is_not_finite(bad):
    """A unit whose score is not positive passes no gradient, so its row of W1 does not reach d_X
    even where it is not finite; a unit with a gradient does; as by lists."""
    gen = torch.Generator(device="cuda").manual_seed(8)
    x, g = (torch.randn(200, 256, generator=gen, device="cuda").bfloat16() for _ in range(2))
    w1, w2 = (torch.randn(500, 256, generator=gen, device="cuda").bfloat16() for _ in range(2))
    assert _ffn_by_cells(200, 256, 500, 128)
    idx = torch.stack([torch.randperm(499, generator=gen, device="cuda")[:128] + 1 for _ in range(200)]).int()
    dots = torch.randn(200, 128, generator=gen, device="cuda")
    dots[idx == 7] = -1.0
    w1[7] = bad
    got = tk.ffn_backward(x, w1, w2, idx, dots, g)
    assert int((idx == 7).any(1).sum()) > 0
    for p, r in zip(got, _lists(lambda: tk.ffn_backward(x, w1, w2, idx, dots, g))):
        assert torch.isfinite(p).all() and torch.isfinite(r).all()
        _close(p, r)
    dots[idx == 7] = 1.0
    got = tk.ffn_backward(x, w1, w2, idx, dots, g)
    lst = _lists(lambda: tk.ffn_backward(x, w1, w2, idx, dots, g))
    assert torch.equal(torch.isfinite(got[0]), torch.isfinite(lst[0]))
    assert torch.equal((~torch.isfinite(got[0])).all(1), (idx == 7).any(1))


def _same_bits(a, b):
    """Equal bit for bit (a NaN's bits included)."""
    return torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("N,dff", [(400, 1000), (140, 4000)])  # whole products, split products
def test_cells_rows_not_finite_repeat(N, dff):
    """Rows computed again because of one column that is not finite: the other columns' sums are the
    same in every call, and near the lists'."""
    gen = torch.Generator(device="cuda").manual_seed(9)
    x, g = (torch.randn(N, 256, generator=gen, device="cuda").bfloat16() for _ in range(2))
    w1, w2 = (torch.randn(dff, 256, generator=gen, device="cuda").bfloat16() for _ in range(2))
    k = 128 if dff == 1000 else 256
    assert _ffn_by_cells(N, 256, dff, k)
    _, idx, dots = tk.ffn(x, w1, w2, k, cache=True)
    w1[:, 3], x[:, 5] = float("inf"), float("inf")
    got = tk.ffn_backward(x, w1, w2, idx, dots, g)
    for _ in range(5):
        for p, q in zip(got, tk.ffn_backward(x, w1, w2, idx, dots, g)):
            assert _same_bits(p, q)
    lst = _lists(lambda: tk.ffn_backward(x, w1, w2, idx, dots, g))
    used = torch.zeros(dff, dtype=torch.bool, device="cuda").index_fill_(0, idx.flatten().long(), True)
    assert not torch.isfinite(got[0][:, 3]).any() and not torch.isfinite(got[1][used, 5]).any()
    for p, r, c in zip(got, lst, (3, 5, 0)):
        keep = torch.arange(256, device="cuda") != c
        _close(p[:, keep], r[:, keep])


@pytest.mark.parametrize("N,dff", [(300, 500), (140, 4000)])  # whole products, split products
def test_cells_keys_listed_often_repeat(N, dff):
    """Keys listed many times in a row: their sums run in pair order, so every call gives the same
    bits; near the lists'."""
    gen = torch.Generator(device="cuda").manual_seed(10)
    x, g = (torch.randn(N, 256, generator=gen, device="cuda").bfloat16() for _ in range(2))
    w1, w2 = (torch.randn(dff, 256, generator=gen, device="cuda").bfloat16() for _ in range(2))
    k = 128 if dff == 500 else 256
    assert _ffn_by_cells(N, 256, dff, k)
    idx = torch.randint(-1, 30, (N, k), generator=gen, device="cuda", dtype=torch.int32)
    idx[:, k // 2:] += dff - 30
    dots = torch.randn(N, k, generator=gen, device="cuda")
    got = tk.ffn_backward(x, w1, w2, idx, dots, g)
    for _ in range(5):
        for p, q in zip(got, tk.ffn_backward(x, w1, w2, idx, dots, g)):
            assert torch.equal(p, q)
    for p, r in zip(got, _lists(lambda: tk.ffn_backward(x, w1, w2, idx, dots, g))):
        _close(p, r)


def test_cells_leave_more_strips_than_a_launch_holds_to_the_lists():
    """2^22 heads of one row are more strips of 1024 threads than a launch can hold. One key per row:
    its weight is 1, whatever its score."""
    B, H = 2048, 2052
    q = torch.ones(B, H, 1, 64, device="cuda", dtype=torch.bfloat16)
    g = torch.randn(B, H, 1, 64, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda").bfloat16()
    idx = torch.zeros(B, H, 1, 1, dtype=torch.int32, device="cuda")
    dq, dk, dv = tk.attn_backward(q, q, q, idx, idx.float(), g)
    assert torch.equal(dv, g) and not dq.any() and not dk.any()
