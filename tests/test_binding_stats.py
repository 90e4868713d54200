"""The statistics' calls through the binding's compiled part and through Python: the same results in the caller's own buffers or new
ones, the same refusals."""
import sys
import types

import pytest
import torch

import paper_2511_04214_amd as brq


def test_left_to_python():
    brq.lib()
    n, x = brq._native, torch.zeros((4, 512))
    assert n.block_stats(x, 32, (1.5,), None, None, True, True, None, None) is None
    assert n.block_stats_summary(x, None, None, 0.0, (), None, None, None) is None
    assert n.block_stats() is None and n.block_stats_summary(None) is None
    with pytest.raises(TypeError):
        n.bind_stats(1)
    with pytest.raises(ValueError):
        n.bind_stats(0, 0)


def test_the_library_does_without_a_compiled_part_built_before_these_calls(monkeypatch):
    brq.lib()
    older = types.SimpleNamespace(TORCH=str(torch.__version__), bind=lambda *a: None)
    monkeypatch.setattr(brq, "_lib", None)
    monkeypatch.setattr(brq, "_native", None)
    monkeypatch.setattr(brq, "_binding", older, raising=False)
    monkeypatch.setitem(sys.modules, brq.__name__ + "._binding", older)
    with pytest.warns(RuntimeWarning, match="compiled part"):
        brq.lib()
    assert brq._native is None and brq.operand_bytes(64, 512) == (16384, 1024)


@pytest.mark.gpu
def test_both_ways_agree():
    s = torch.cuda.current_stream()                     # (a Stream argument takes the way through Python)
    g = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn((37, 2 * 736), generator=g, device="cuda").to(torch.bfloat16)[:, :736]
    signs = (torch.randint(0, 2, (736,), generator=g, device="cuda") * 2 - 1).to(torch.int8)
    new = lambda: (torch.full((37, 23), -1.0, device="cuda"), torch.full((37, 23), -1.0, device="cuda"), torch.ones((2,), dtype=torch.int64, device="cuda"))
    for kw in (dict(), dict(thresholds=(1.5, 3)), dict(thresholds=[1.5] * 8, signs=signs), dict(want_sqerr=False), dict(want_amax=False, thresholds=(0.5,))):
        a, b = brq.block_stats(x, 32, **kw), brq.block_stats(x, 32, stream=s, **kw)
        assert type(a) is tuple and len(a) == 3
        for u, v in zip(a, b):
            assert (u is None and v is None) or (u.dtype == v.dtype and torch.equal(u, v))
    given = [new(), new()]
    for (am, sq, c), kw in zip(given, (dict(), dict(stream=s))):
        r = brq.block_stats(x, 1, (1.0, 2.0), None, c, False, False, amax=am, sqerr=sq, **kw)
        assert r[0] is am and r[1] is c and r[2] is sq
    for u, v in zip(*given):
        assert torch.equal(u, v)
    am, c, sq = brq.block_stats(x, 32, thresholds=(1.0,))
    ref = brq.block_stats(x, 1)[0]
    for kw in (dict(), dict(sqerr=sq, amax_ref=ref, outlier_threshold=2, edges=(0.5, 1, 2.0)), dict(amax_ref=ref, edges=[1.0] * 32)):
        a, b = brq.block_stats_summary(am, **kw), brq.block_stats_summary(am, stream=s, **kw)
        assert type(a) is tuple and all(u.dtype == v.dtype and torch.equal(u, v) for u, v in zip(a[:2], b[:2]))
        assert a[2].dtype == torch.float64 and torch.allclose(a[2], b[2], rtol=1e-12, atol=0)      # (sums by atomics, in any order)
        assert all(u.is_contiguous() and u.untyped_storage().nbytes() == u.numel() * 8 for u in a)
    h, k = torch.ones((2,), dtype=torch.int64, device="cuda"), torch.ones((4,), dtype=torch.int64, device="cuda")
    r = brq.block_stats_summary(am, edges=(1.0,), hist=h, counts=k)
    assert r[0] is h and r[1] is k and int(h.sum()) == am.numel() + 2


@pytest.mark.gpu
def test_what_is_refused_stays_refused():
    x = torch.zeros((4, 512), device="cuda")
    c = torch.zeros((1,), dtype=torch.int64, device="cuda")
    for call, err in ((lambda: brq.block_stats(x, 33), brq.BrqError), (lambda: brq.block_stats(x[:, :500], 32), brq.BrqError),
                      (lambda: brq.block_stats(x, 32, thresholds=[1.0] * 9), brq.BrqError), (lambda: brq.block_stats(x.t(), 32), ValueError),
                      (lambda: brq.block_stats(x, 32, thresholds=(1.0, 2.0), counts=c), ValueError), (lambda: brq.block_stats(x.half(), 32), TypeError),
                      (lambda: brq.block_stats(x, 32, amax=torch.zeros((4, 15), device="cuda")), ValueError),
                      (lambda: brq.block_stats(x, 32, signs=torch.ones((511,), dtype=torch.int8, device="cuda")), ValueError),
                      (lambda: brq.block_stats(x.cpu(), 32), ValueError), (lambda: brq.block_stats_summary(x.t()), ValueError),
                      (lambda: brq.block_stats_summary(x, sqerr=x[:2]), ValueError), (lambda: brq.block_stats_summary(x, edges=(2.0, 1.0)), brq.BrqError),
                      (lambda: brq.block_stats_summary(x, edges=(1.0,), hist=c), ValueError)):
        with pytest.raises(err):
            call()
