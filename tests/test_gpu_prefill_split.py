"""GPU prefill with its key tiles shared evenly over the chip
(jf_prefill_attn_q4_ws) against the CPU oracle and against the call that keeps
row blocks whole (jf_prefill_attn_q4), at shapes whose shares end inside a row
block, on its edge, and span several row blocks, with last tiles that are
partial, waves without rows, and a page outside the pool.

Both calls run the same products per tile; only the fp32 sums over tiles are
taken in another order (and relative to another running maximum, so p is
rounded to fp16 at another scale, at most 2^-11 relative each).  Both hold the
oracle's tolerance of test_gpu_prefill, 2e-3 + 2^-11 |o| elementwise and 1e-3
in relative L2, so they are at most twice that apart."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2609_17475_amd import jfkv


def test_prefill_workspace_bytes_and_validation():
    lay = jfkv.layout(256, 8, 128, 64, 16)
    # the state of a 256-row block: o, and m and l for each of a row's four lanes
    part = 256 * (128 + 4 * 2) * 4
    # a full chunk of whole turns without a prefix worth sharing needs none
    assert jfkv.jf_prefill_workspace_bytes(lay, 0, 32, 0) == 0
    assert jfkv.jf_prefill_workspace_bytes(lay, 64, 32, 0) == 0
    # bounded by two states per compute unit, whatever the lengths
    for T, p0 in ((20, 3000), (256, 200000), (1000, 7000), (2049, 65536)):
        n = jfkv.jf_prefill_workspace_bytes(lay, T, 32, p0)
        assert 0 < n <= 2 * 256 * part and n % part == 0
    # ... of 256 rows at head_dim 64 and 128 rows at 256
    for d, part, mb in ((64, 256 * (64 + 8) * 4, 38), (128, part, 72), (256, 128 * (256 + 8) * 4, 70)):
        n = jfkv.jf_prefill_workspace_bytes(jfkv.layout(256, 4, d, 64, 16), 300, 24, 200000)
        assert 0 < n <= 2 * 256 * part <= mb * 10 ** 6 and n % part == 0
    with pytest.raises(jfkv.JfError):
        jfkv.jf_prefill_workspace_bytes(lay, 64, 30, 0)
    ptrs = jfkv.PoolPtrs(1, 1, 1, 1)
    call = jfkv.lib.jf_prefill_attn_q4_ws
    for ws, n in ((None, 1 << 40), (16, 100), (8, 1 << 40)):
        assert call(ctypes.byref(lay), ctypes.byref(ptrs), 1, 1, 1, 20, 32, 1, 16, 3000, 1.0, ws, n,
                    1, None) == jfkv.JF_ERR_INVALID
        assert b"workspace" in jfkv.lib.jf_last_error()


@pytest.mark.gpu
@pytest.mark.parametrize("P,hkv,hq,d,G,p0,T,scale,bad", [
    (256, 1, 4, 128, 64, 5000, 37, 1.0, None),    # one row block, waves without rows
    (64, 2, 8, 128, 32, 3001, 130, -0.7, None),   # three row blocks, partial last tiles
    (256, 1, 8, 128, 128, 2048, 64, 1.0, 3),      # whole pages, one outside the pool
    (64, 1, 2, 64, 64, 2111, 300, 1.0, None),
    (256, 4, 24, 256, 64, 1500, 50, 1.0, None),   # 32-key tiles
    (64, 1, 16, 256, 32, 900, 29, 1.3, 5),
    (64, 1, 4, 128, 64, 0, 1700, 1.0, None),      # shares over several short row blocks
])
def test_split_prefill_matches_oracle_and_whole_row_blocks(P, hkv, hq, d, G, p0, T, scale, bad):
    import oracle
    from gpu_cases import build, check_tol, log
    log("split prefill P=%d hkv=%d hq=%d d=%d G=%d p0=%d T=%d scale=%g bad=%s" % (
        P, hkv, hq, d, G, p0, T, scale, bad))
    case = build(P=P, hkv=hkv, d=d, G=G, hq=hq, lens=(p0 + T,), n_out=2, seed=p0 + T)
    rng = np.random.default_rng(p0 * 5 + T)
    kc = rng.standard_normal((T, hkv, d)).astype(np.float16)
    vc = rng.standard_normal((T, hkv, d)).astype(np.float16)
    q = (rng.standard_normal((T, hq, d)) / np.sqrt(d)).astype(np.float16)
    table = np.ascontiguousarray(case.tables[0])
    if bad is not None:
        table[bad] = case.lay.num_pages + 7
    nbytes = jfkv.jf_prefill_workspace_bytes(case.lay, T, hq, p0)
    assert nbytes > 0
    args = [torch.from_numpy(x).cuda() for x in (q, kc, vc, table)]
    split = torch.full(q.shape, float("nan"), dtype=torch.float16, device="cuda")
    whole = split.clone()
    # the binding takes the workspace by itself; poison what it may be given
    torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
    jfkv.jf_prefill_attn_q4(case.gpu, *args, p0, scale, split)
    bound = torch.full_like(split, float("nan"))
    jfkv.bind_prefill(case.gpu, *args, p0, scale, bound)()
    lay, ptrs = case.lay, case.gpu.ptrs()
    jfkv._check(jfkv.lib.jf_prefill_attn_q4(
        ctypes.byref(lay), ctypes.byref(ptrs), *(a.data_ptr() for a in args[:3]), T, hq,
        args[3].data_ptr(), len(table), p0, scale, whole.data_ptr(),
        torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert torch.equal(split, bound)
    tol = dict(atol=2e-3, rel_elem=2.0 ** -11, rel_l2=1e-3)
    check_tol(split.cpu().numpy(), whole.double().cpu().numpy(), what="split against whole",
              **{k: 2 * v for k, v in tol.items()})
    if bad is not None:  # (the oracle takes no page outside the pool)
        return
    ref = oracle.prefill(case.host, q, kc, vc, table, p0, scale)
    log("  max err %.3e rel L2 %.3e" % check_tol(split.cpu().numpy(), ref, what="split", **tol))


def _layout(hkv, hq, d, G, p0, T):
    """Blocks per KV head and row blocks of a call (0 blocks: not split)."""
    rows = 128 if d == 256 else 256
    part = rows * (d + 4 * 2) * 4
    n = jfkv.jf_prefill_workspace_bytes(jfkv.layout(64, hkv, d, G, 64), T, hq, p0)
    return n // (2 * hkv * part), -(-T * (hq // hkv) // rows)


@pytest.mark.gpu
@pytest.mark.parametrize("P,hkv,hq,d,G,p0,T,form", [
    # few parts per row block (the combine's first form), some (its second)
    (64, 64, 64, 64, 32, 1500, 400, 1),
    (64, 32, 64, 128, 32, 300, 390, 1),
    (64, 8, 16, 256, 32, 200, 1100, 1),
    (64, 2, 8, 64, 64, 700, 300, 2),
    (64, 4, 8, 256, 64, 500, 300, 2),
    # more row blocks than blocks: shares hold whole row blocks, whose rows are
    # written by the block itself in the middle of a split call
    (64, 32, 64, 64, 32, 400, 1100, 0),
    (64, 32, 64, 256, 64, 400, 520, 0),
    # no prefix, split and whole, odd numbers of rows
    (64, 2, 8, 64, 32, 0, 1101, 1),
    (64, 8, 8, 64, 64, 0, 1201, 1),
    (64, 4, 8, 256, 64, 0, 701, 2),
    (64, 1, 4, 256, 128, 0, 901, 2),
    (64, 1, 4, 128, 32, 0, 1301, 1),
    (64, 2, 8, 64, 64, 0, 151, None),
    (64, 1, 2, 64, 32, 0, 65, None),
    (64, 4, 24, 256, 64, 0, 101, None),
    (64, 2, 8, 256, 32, 0, 77, None),
])
def test_split_prefill_forms_match_oracle(P, hkv, hq, d, G, p0, T, form):
    """Every form of the split call and its combine at every head size, all rows
    against the oracle.  form: 1 and 2, up to 4 and up to 16 parts per row block;
    0, more row blocks than blocks; None, not split.

    Tolerance: p is rounded to fp16, 2^-11 of itself at most, so an output moves
    by at most 2^-11 sum p |v - o| beside its own rounding, 2^-11 |o|.  The values
    are unit normals (no outlier channels: with those, |v - o| up to ~24, one of
    the 1.6 million outputs of the first case is 5.6e-3 off, split or whole);
    their mean distance from a weighted mean is below 2: 1e-3."""
    import oracle
    from gpu_cases import build, check_tol, log
    n_blk, n_rb = _layout(hkv, hq, d, G, p0, T)
    log("split prefill hkv=%d hq=%d d=%d G=%d p0=%d T=%d: %d blocks, %d row blocks" % (
        hkv, hq, d, G, p0, T, n_blk, n_rb))
    parts = n_blk // n_rb + 2
    assert {None: n_blk == 0, 0: 0 < n_blk < n_rb, 1: n_blk >= n_rb and parts <= 4, 2: 4 < parts <= 16}[form]
    case = build(P=P, hkv=hkv, d=d, G=G, hq=hq, lens=(p0 + T,), n_out=0, seed=p0 + T)
    rng = np.random.default_rng(p0 * 3 + T)
    kc, vc = (rng.standard_normal((T, hkv, d)).astype(np.float16) for _ in range(2))
    q = (rng.standard_normal((T, hq, d)) / np.sqrt(d)).astype(np.float16)
    args = [torch.from_numpy(x).cuda() for x in (q, kc, vc, case.tables[0])]
    out = torch.full(q.shape, float("nan"), dtype=torch.float16, device="cuda")
    jfkv.jf_prefill_attn_q4(case.gpu, *args, p0, 1.0, out)
    torch.cuda.synchronize()
    ref = oracle.prefill(case.host, q, kc, vc, case.tables[0], p0, 1.0)
    log("  max err %.3e rel L2 %.3e" % check_tol(out.cpu().numpy(), ref, atol=1e-3, rel_elem=2.0 ** -11,
                                                 rel_l2=1e-3, what="split"))


def _call(P, hkv, hq, d, G, p0, T):
    """A split call: its pool and arguments, its workspace's bytes, and what the
    split call and the call of whole row blocks give."""
    from gpu_cases import build
    case = build(P=P, hkv=hkv, d=d, G=G, hq=hq, lens=(p0 + T,), seed=p0 + T)
    g = torch.Generator(device="cuda").manual_seed(T)
    q, kc, vc = (torch.randn((T, h, d), generator=g, device="cuda").half() for h in (hq, hkv, hkv))
    args = (case.gpu, q, kc, vc, torch.from_numpy(case.tables[0]).cuda(), p0, d ** -0.5)
    nbytes = jfkv.jf_prefill_workspace_bytes(case.lay, T, hq, p0)
    assert nbytes > 0
    split, whole = (torch.full_like(q, float("nan")) for _ in range(2))
    jfkv.jf_prefill_attn_q4(*args, split)
    lay, ptrs = case.lay, case.gpu.ptrs()
    jfkv._check(jfkv.lib.jf_prefill_attn_q4(
        ctypes.byref(lay), ctypes.byref(ptrs), *(a.data_ptr() for a in args[1:4]), T, hq,
        args[4].data_ptr(), len(args[4]), p0, args[6], whole.data_ptr(),
        torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert not torch.equal(split, whole)  # (sums in another order: the layouts can be told apart)
    return args, nbytes, split, whole


@pytest.mark.gpu
def test_callers_workspace_eager_and_captured():
    """With the caller's workspace a call is split as it is without, eagerly and
    in a graph, to the bit; a captured call without one keeps row blocks whole."""
    from gpu_cases import log
    log("prefill with the caller's workspace, captured")
    args, nbytes, split, whole = _call(256, 1, 4, 128, 64, 5000, 37)
    ws = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
    out = torch.full_like(split, float("nan"))
    jfkv.jf_prefill_attn_q4(*args, out, workspace=ws)
    assert torch.equal(out, split)
    out.fill_(float("nan"))
    jfkv.bind_prefill(*args, out, workspace=ws)()
    assert torch.equal(out, split)
    for short in (ws[:nbytes - 16], ws[8:]):  # too small, misaligned
        with pytest.raises(jfkv.JfError, match="workspace"):
            jfkv.jf_prefill_attn_q4(*args, out, workspace=short)
    with pytest.raises(ValueError, match="workspace"):
        jfkv.jf_prefill_attn_q4(*args, out, workspace=ws.cpu())

    out2, out3 = torch.full_like(split, float("nan")), torch.full_like(split, float("nan"))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        jfkv.bind_prefill(*args, out, workspace=ws)()
        jfkv.jf_prefill_attn_q4(*args, out2)
        jfkv.bind_prefill(*args, out3)()
    for _ in range(3):
        for t in (out, out2, out3):
            t.fill_(float("nan"))
        ws.fill_(0xA5)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, split) and torch.equal(out2, whole) and torch.equal(out3, whole)
        eager = torch.full_like(split, float("nan"))
        jfkv.jf_prefill_attn_q4(*args, eager)
        assert torch.equal(eager, split)


@pytest.mark.gpu
def test_other_streams_and_no_memory(monkeypatch):
    from types import SimpleNamespace

    from gpu_cases import log
    log("split prefill on other streams, without scratch")
    args, nbytes, split, whole = _call(64, 2, 8, 128, 32, 3001, 130)
    side = torch.cuda.Stream()
    for stream in (side, SimpleNamespace(cuda_stream=side.cuda_stream)):
        out = torch.full_like(split, float("nan"))
        torch.cuda.synchronize()
        jfkv.jf_prefill_attn_q4(*args, out, stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(out, split)
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        jfkv.bind_prefill(*args, out, stream=stream)()
        torch.cuda.synchronize()
        assert torch.equal(out, split)
    out = torch.full_like(split, float("nan"))

    def no_memory(*_, **__):
        raise torch.OutOfMemoryError("no memory")

    monkeypatch.setattr(torch, "empty", no_memory)
    jfkv.jf_prefill_attn_q4(*args, out)
    torch.cuda.synchronize()
    monkeypatch.undo()
    assert torch.equal(out, whole)
