"""GPU tests of the few-query kernels (at most 128 bf16 queries per head, 1025 to 65536
keys): against the fp64 oracle at the edges of their row groups, key blocks and lists,
with equal scores (the fallback), and independent of the chunk size; and of the finalize
that gives few rows eight waves each."""
import numpy as np
import pytest
import torch

import paper_2106_06899_amd as tk
from paper_2106_06899_amd import workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu

# (B, H, Lq, Lk, d, k): row groups of 16, 32 and 64; ragged 16-key blocks; 16 and 64 keys a
# wave; block lists of 8 to 64 per lane; features beyond one step; k around the list sizes
CASES = [(1, 1, 1, 1025, 64, 1), (1, 3, 16, 1040, 128, 50), (2, 2, 17, 2047, 32, 52), (1, 2, 32, 9000, 64, 128),
         (2, 16, 33, 4099, 128, 64), (1, 8, 64, 20001, 96, 256), (1, 1, 65, 33000, 64, 257), (1, 2, 128, 16000, 160, 512),
         (1, 2, 5, 65536, 1024, 512), (1, 4, 3, 10244, 544, 512)]


@pytest.mark.parametrize("case", CASES)
def test_few_queries(case):
    B, H, Lq, Lk, d, k = case
    w = wl.WORKLOADS["c2"].scaled(B=B, H=H, Lq=Lq, Lk=Lk, d=d, k=k, chunk=1024, scale=float(np.float32(d ** -0.5)))
    print("[case]", w, flush=True)
    assert tk.attn_path(B, H, Lq, Lk, d, k, w.chunk, False) == 2
    x = wl.make_inputs(w)
    out, idx, sc = parity.run_attn(w, x)
    assert tk.last_fallback_rows() == 0
    parity.check_attn(w, x, out, idx, rows=parity.sample_attn_rows(w, min(B * H * Lq, 60), seed=3))
    g = idx.cpu().numpy().reshape(-1, k)
    assert np.all(np.diff(np.sort(g, axis=1), axis=1) > 0) and g.min() >= 0 and g.max() < Lk
    assert torch.equal(parity.run_attn(w, x, debug=False), out)


@pytest.mark.parametrize("band", [0.0, 1e-30])
def test_few_queries_equal_scores(band):
    """Equal scores (or all below the smallest normal number apart): every block reaches
    the bound, the rows are settled by the fallback, and the lowest indices are kept."""
    w = wl.WORKLOADS["c2"].scaled(B=1, H=2, Lq=7, Lk=20000, k=64)
    x = wl.make_inputs(w)
    x["Q"] = wl._store((x["Q"].values * np.float32(band)).astype(np.float32), w.dtype)
    print("[case] equal scores", band, w, flush=True)
    out, idx, _ = parity.run_attn(w, x)
    parity.check_attn(w, x, out, idx)
    if band == 0.0:
        assert tk.last_fallback_rows() == 14
        assert torch.equal(idx.cpu(), torch.arange(64, dtype=torch.int32).expand(1, 2, 7, 64))


def test_few_queries_any_chunk_and_the_fixed_scratch():
    w = wl.WORKLOADS["c3"].scaled(H=4, Lq=40, Lk=20000, chunk=1024)
    x = wl.make_inputs(w)
    ref = parity.run_attn(w, x)
    for C in (1, 7, 32):
        print("[case] chunk", C, flush=True)
        assert tk.attn_path(w.B, w.H, w.Lq, w.Lk, w.d, w.k, C, False) == 2
        for a, b in zip(ref, parity.run_attn(w, x, chunk=C)):
            assert torch.equal(a, b)
    tk.set_memory_budget(1)  # one head per pass
    try:
        for a, b in zip(ref, parity.run_attn(w, x)):
            assert torch.equal(a, b)
    finally:
        tk.set_memory_budget(0)
    q, k, v = (parity.to_dev(x[n]) for n in ("Q", "K", "V"))
    got = torch.empty_like(q)
    tk._raise(tk.lib().topk_attn_noalloc(q.data_ptr(), k.data_ptr(), v.data_ptr(), got.data_ptr(), w.B, w.H, w.Lq, w.Lk, w.d, w.k,
                                         w.chunk, 0, w.scale, tk.TOPK_BF16, torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert torch.equal(got, ref[0])


@pytest.mark.parametrize("kw", [
    dict(N=1, d_model=8, d_ff=2000, k=3), dict(N=128, d_model=96, d_ff=2048, k=512), dict(N=129, d_model=72, d_ff=1500, k=700),
    dict(N=512, d_model=256, d_ff=3000, k=128), dict(N=24, d_model=768, d_ff=5000, k=256),
    dict(N=60, d_model=200, d_ff=1100, k=2, dtype=wl.F32), dict(N=300, d_model=1024, d_ff=1500, k=1000, dtype=wl.F32)])
def test_finalize_of_few_rows(kw):
    """Column slices of 128 bytes (partial last ones), fewer and more survivors than the 64
    row slots, in both types."""
    w = wl.WORKLOADS["c5"].scaled(chunk=50, **kw)
    print("[case]", w, flush=True)
    x = wl.make_inputs(w)
    out, idx, _ = parity.run_ffn(w, x)
    parity.check_ffn(w, x, out, idx)
    assert torch.equal(parity.run_ffn(w, x, debug=False), out)


@pytest.mark.parametrize("Lk,d,k", [(1800, 64, 85), (1030, 96, 40), (2048, 160, 64), (1999, 128, 90)])
def test_few_queries_in_chunks_of_the_tile_path(Lk, d, k):
    """Where they take the place of the chunk-tile path the kernels run chunk by chunk: the same kernel
    whatever the chunk size (its workspace holds the block maxima), and the same bits; in a workspace
    too small for the maxima, the chunk-tile path's own kernels."""
    w = wl.WORKLOADS["c2"].scaled(B=2, H=3, Lq=100, Lk=Lk, d=d, k=k, chunk=128, scale=float(np.float32(d ** -0.5)))
    x = wl.make_inputs(w)
    ref = parity.run_attn(w, x)
    parity.check_attn(w, x, ref[0], ref[1], rows=parity.sample_attn_rows(w, 60, seed=3))
    for C in (1, 7, 33, 64, 100):
        print("[case] chunk", C, w, flush=True)
        assert tk.attn_workspace_bytes(w.B, w.H, w.Lq, Lk, d, k, C) >= w.B * w.H * w.Lq * ((Lk + 15) // 16 * 68 + 8 * k)
        for a, b in zip(ref, parity.run_attn(w, x, chunk=C)):
            assert torch.equal(a, b)
    q, kk, v = (parity.to_dev(x[n]) for n in ("Q", "K", "V"))
    got = torch.empty_like(q)
    size = 100 * (4 * Lk + 8 * k + 4) + 8 * 256  # one chunk of the chunk-tile path
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    tk._raise(tk.lib().topk_set_workspace(ws.data_ptr(), size))
    try:
        tk._raise(tk.lib().topk_attn(q.data_ptr(), kk.data_ptr(), v.data_ptr(), got.data_ptr(), w.B, w.H, w.Lq, Lk, d, k, 100, 0,
                                     w.scale, tk.TOPK_BF16, torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
    finally:
        tk.lib().topk_set_workspace(None, 0)
    parity.check_attn(w, x, got, ref[1], rows=parity.sample_attn_rows(w, 60, seed=3))


@pytest.mark.parametrize("score_only", [False, True])
def test_scan_ablation_of_few_queries(score_only):
    """The measurement hook times the scan at any number of queries."""
    gen = torch.Generator(device="cuda").manual_seed(1)
    q, k = (torch.randn(1, 4, n, 64, generator=gen, device="cuda").bfloat16() for n in (100, 20000))
    tk.profile_begin()
    tk.scan_ablation(q, k, 64, score_only=score_only)
    assert tk.profile_end()["score"][1] == 1


# (heads, Lq, Lk, d, k): fewer, as many and more 16-key blocks than k; the smallest and largest
# rows; more rows than the few-query kernels take (the last: chunk tiles)
SHORT = [(410, 1, 1024, 128, 20), (830, 2, 1000, 64, 63), (412, 3, 1023, 128, 64), (820, 8, 1024, 64, 65), (1700, 1, 300, 128, 256),
         (6400, 1, 257, 32, 17), (3280, 4, 257, 64, 200), (1100, 8, 520, 96, 100)]


@pytest.mark.parametrize("case", SHORT)
def test_few_queries_against_many_short_rows(case):
    """Heads of at most 1024 keys whose keys and values together exceed the caches: a handful of
    queries takes the general paths, more queries or fewer heads the short-row kernel (256 bytes
    of workspace). Against 64 bits."""
    H, Lq, Lk, d, k = case
    print("[case]", case, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, kk, v = (torch.randn(1, H, n, d, generator=gen, device="cuda").bfloat16() for n in (Lq, Lk, Lk))
    assert tk.attn_path(1, H, Lq, Lk, d, k) == 2 and tk.attn_workspace_bytes(1, H, Lq, Lk, d, k) > 256
    assert tk.attn_workspace_bytes(1, H, 9, Lk, d, k) == 256 and tk.attn_workspace_bytes(1, H // 2, Lq, Lk, d, k) == 256
    out, idx, sc = tk.attn(q, kk, v, k, debug=True)
    assert tk.last_fallback_rows() == 0
    s = q.double() @ kk.double().transpose(2, 3).contiguous()
    got = s.gather(3, idx.long())
    # 32-bit sums of up to 128 products of size 1: scores this close may swap
    assert bool(((got - s.topk(k, dim=-1).values).abs() <= 1e-4).all()) and bool(((sc.double() - got).abs() <= 1e-4).all())
    assert k == 1 or bool((idx.long().sort(-1).values.diff(dim=-1) > 0).all())
    w = torch.softmax(got * d ** -0.5, -1)
    for h in range(0, H, 64):
        p = torch.zeros_like(s[:, h:h + 64]).scatter_(3, idx[:, h:h + 64].long(), w[:, h:h + 64])
        ref = p @ v[:, h:h + 64].double()
        assert bool(((out[:, h:h + 64].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5).all())
    for C in (1, 3):
        assert torch.equal(tk.attn(q, kk, v, k, C), out)


def test_few_queries_where_the_filtered_path_does_not_fit():
    """More scores than these kernels are the faster for, in the fixed scratch, which the filtered
    path's fallback rows exceed: they run there."""
    H, Lq, Lk, d, k = 1, 100, 45000, 256, 512
    assert tk.attn_path(1, H, Lq, Lk, d, k) == 4 and tk.attn_workspace_bytes(1, H, Lq, Lk, d, k) > tk.lib().topk_noalloc_scratch_bytes()
    gen = torch.Generator(device="cuda").manual_seed(8)
    q, kk, v = (torch.randn(1, H, n, d, generator=gen, device="cuda").bfloat16() for n in (Lq, Lk, Lk))
    ref, got = tk.attn(q, kk, v, k), torch.empty_like(q)
    tk._raise(tk.lib().topk_attn_noalloc(q.data_ptr(), kk.data_ptr(), v.data_ptr(), got.data_ptr(), 1, H, Lq, Lk, d, k, 0, 0, d ** -0.5,
                                         tk.TOPK_BF16, torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    # sums in another order: a result on the other side of a rounding (2^-8)
    assert bool(((got.float() - ref.float()).abs().amax(-1) <= 2.0 ** -7 * ref.float().abs().amax(-1)).all())
