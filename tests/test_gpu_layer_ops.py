"""GPU parity of the dense operators around the attention (cc_rms_norm, cc_linear, cc_gated_linear)
against the oracle, through the C ABI: plain and MFMA kernels, ragged row counts, in-place
residuals, and the layer's tail composed from them."""
import math

import numpy as np
import pytest
import torch

import workload as W
from oracle import cachecraft_oracle as O
from tests import helpers as H

pytestmark = pytest.mark.gpu


def _ctx(dtype, impl="auto"):
    import paper_2502_15734_amd as P
    ctx = P.Context(8, 2, 128, 5.0e5, P.CC_BF16 if dtype == "bf16" else P.CC_F32)
    ctx.set_impl({"auto": P.CC_IMPL_AUTO, "scalar": P.CC_IMPL_SCALAR, "narrow": P.CC_IMPL_MFMA_NARROW,
                  "wide": P.CC_IMPL_MFMA_WIDE}[impl])
    return ctx


def _dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a)).to(torch.bfloat16 if dtype == "bf16" else torch.float32).cuda()


def _draw(rng, shape, scale, dtype):
    a = (rng.standard_normal(shape) * scale).astype(np.float32)
    return W.round_to_bf16(a) if dtype == "bf16" else a


def _host(t):
    return t.float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("dtype,rows,hidden", [("bf16", 1, 256), ("bf16", 37, 4096), ("bf16", 301, 40),
                                               ("f32", 5, 36), ("f32", 130, 1024), ("bf16", 9, 8192),
                                               ("bf16", 3, 16384), ("f32", 6, 8192)])   # rows kept in registers / read twice
def test_rms_norm(dtype, rows, hidden):
    rng = np.random.default_rng(rows + hidden)
    x = _draw(rng, (rows, hidden), 1.5, dtype)
    x[0] *= 1e-3                                                      # a row whose mean square is close to eps
    g = _draw(rng, (hidden,), 0.1, dtype) + np.float32(1.0)
    g = W.round_to_bf16(g) if dtype == "bf16" else g
    ctx = _ctx(dtype)
    xd, gd = _dev(x, dtype), _dev(g, dtype)
    yd = torch.full_like(xd, float("nan"))
    ctx.rms_norm(xd, gd, 1e-5, yd); torch.cuda.synchronize()
    want = O.rms_norm(x, g, 1e-5)
    assert H.rel_l2(_host(yd), want) <= H.TOL[dtype]
    assert np.abs(_host(yd) - want).max() <= (2e-2 if dtype == "bf16" else 1e-5) * max(1.0, np.abs(want).max())
    ctx.rms_norm(xd, gd, 1e-5, xd); torch.cuda.synchronize()         # in place
    assert torch.equal(xd, yd)
    ctx.close()


LINEAR_CASES = [("f32", "auto", 37, 40, 50), ("f32", "auto", 130, 64, 256), ("bf16", "auto", 300, 256, 512),
                ("bf16", "auto", 256, 96, 256), ("bf16", "auto", 41, 72, 40), ("bf16", "scalar", 70, 256, 256),
                ("bf16", "narrow", 70, 256, 256), ("bf16", "wide", 513, 1024, 768),
                ("bf16", "auto", 1, 64, 256), ("bf16", "auto", 257, 128, 256),      # one and two 64-wide stages
                ("bf16", "auto", 2300, 192, 1280)]                                  # tile blocks with ragged edges


@pytest.mark.parametrize("dtype,impl,rows,n_in,n_out", LINEAR_CASES)
def test_linear_with_and_without_residual(dtype, impl, rows, n_in, n_out):
    rng = np.random.default_rng(rows * 7 + n_in)
    x = _draw(rng, (rows, n_in), 1.0, dtype)
    w = _draw(rng, (n_out, n_in), 1.0 / math.sqrt(n_in), dtype)
    res = _draw(rng, (rows, n_out), 1.0, dtype)
    ctx = _ctx(dtype, impl)
    xd, wd, rd = _dev(x, dtype), _dev(w, dtype), _dev(res, dtype)
    yd = torch.full((rows, n_out), float("nan"), dtype=xd.dtype, device="cuda")
    ctx.linear(xd, wd, yd); torch.cuda.synchronize()
    assert H.rel_l2(_host(yd), O.linear(x, w)) <= H.TOL[dtype]
    ctx.linear(xd, wd, yd, residual=rd); torch.cuda.synchronize()
    want = res.astype(np.float64) + O.linear(x, w)
    assert H.rel_l2(_host(yd), want) <= H.TOL[dtype]
    first = yd.clone()
    ctx.linear(xd, wd, rd, residual=rd); torch.cuda.synchronize()     # accumulate into the residual itself
    assert torch.equal(rd, first)
    ctx.close()


GATED_CASES = [("f32", "auto", 37, 40, 50), ("bf16", "auto", 300, 256, 384), ("bf16", "auto", 41, 72, 40),
               ("bf16", "scalar", 70, 256, 128), ("bf16", "wide", 513, 512, 640), ("bf16", "auto", 5, 64, 128)]


@pytest.mark.parametrize("dtype,impl,rows,n_in,n_ffn", GATED_CASES)
def test_gated_linear(dtype, impl, rows, n_in, n_ffn):
    rng = np.random.default_rng(rows * 11 + n_ffn)
    x = _draw(rng, (rows, n_in), 1.0, dtype)
    wg = _draw(rng, (n_ffn, n_in), 2.0 / math.sqrt(n_in), dtype)      # gates on both sides of the SiLU's bend
    wu = _draw(rng, (n_ffn, n_in), 1.0 / math.sqrt(n_in), dtype)
    ctx = _ctx(dtype, impl)
    yd = torch.full((rows, n_ffn), float("nan"), dtype=_dev(x, dtype).dtype, device="cuda")
    ctx.gated_linear(_dev(x, dtype), _dev(wg, dtype), _dev(wu, dtype), yd); torch.cuda.synchronize()
    want = O.gated_ffn_in(x, wg, wu)
    assert H.rel_l2(_host(yd), want) <= H.TOL[dtype]
    assert np.abs(_host(yd) - want).max() <= (3e-2 if dtype == "bf16" else 1e-5) * max(1.0, np.abs(want).max())
    ctx.close()


def _tail_on_gpu(ctx, lw, h, o, dtype):
    hd, od = _dev(h, dtype), _dev(o.reshape(o.shape[0], -1), dtype)
    h1 = torch.empty_like(hd); y = torch.empty_like(hd); h2 = torch.empty_like(hd)
    act = torch.empty((h.shape[0], lw.w_gate.shape[0]), dtype=hd.dtype, device="cuda")
    ctx.linear(od, _dev(lw.w_o, dtype), h1, residual=hd)
    ctx.rms_norm(h1, _dev(lw.gain_ffn, dtype), lw.eps, y)
    ctx.gated_linear(y, _dev(lw.w_gate, dtype), _dev(lw.w_up, dtype), act)
    ctx.linear(act, _dev(lw.w_down, dtype), h2, residual=h1)
    torch.cuda.synchronize()
    return _host(h1), _host(h2)


@pytest.mark.parametrize("dtype,rows,hidden,ffn", [("f32", 45, 64, 160), ("bf16", 333, 256, 640)])
def test_layer_tail_composed_from_the_calls(dtype, rows, hidden, ffn):
    spec = W.config_spec(2)
    spec.dtype = dtype
    lw = W.layer_weights(spec, hidden, ffn)
    rng = np.random.default_rng(rows)
    h = _draw(rng, (rows, hidden), 1.0, dtype)
    o = _draw(rng, (rows, spec.n_q_heads, spec.head_dim), 0.5, dtype)
    ctx = _ctx(dtype)
    h1, h2 = _tail_on_gpu(ctx, lw, h, o, dtype)
    w1, w2 = O.layer_tail(h, o, lw.w_o, lw.gain_ffn, lw.w_gate, lw.w_up, lw.w_down, lw.eps)
    assert H.rel_l2(h1, w1) <= H.TOL[dtype] and H.rel_l2(h2, w2) <= H.TOL[dtype]
    ctx.close()


def test_layer_tail_at_the_8b_model_shape_on_sampled_rows():
    """hidden 4096, feed-forward 14336, 32 heads of 128: the MFMA kernels on several full tiles and a
    ragged one; the oracle follows on sampled rows (a row depends on no other row)."""
    spec = W.config_spec(3)
    hidden, ffn, rows = 4096, 14336, 1000
    lw = W.layer_weights(spec, hidden, ffn)
    rng = np.random.default_rng(3)
    h = _draw(rng, (rows, hidden), 1.0, "bf16")
    o = _draw(rng, (rows, spec.n_q_heads, spec.head_dim), 0.5, "bf16")
    ctx = _ctx("bf16")
    h1, h2 = _tail_on_gpu(ctx, lw, h, o, "bf16")
    which = np.array([0, 127, 128, 255, 256, 511, 777, 999])
    w1, w2 = O.layer_tail(h[which], o[which], lw.w_o, lw.gain_ffn, lw.w_gate, lw.w_up, lw.w_down, lw.eps)
    assert H.rel_l2(h1[which], w1) <= 1e-2 and H.rel_l2(h2[which], w2) <= 1e-2
    assert np.isfinite(h2).all()
    ctx.close()


def _products_in_parts():
    """Context, tensors and a call of a QKV projection and a linear product whose contractions run in parts."""
    import paper_2502_15734_amd as P
    g = torch.Generator(device="cuda").manual_seed(7)
    rnd = lambda *shape, sc=1.0: (torch.randn(*shape, device="cuda", generator=g) * sc).to(torch.bfloat16)
    ctx = P.Context(8, 2, 128, 5.0e5, P.CC_BF16)
    x, w_qkv, a, w_down = rnd(100, 4096), rnd(1536, 4096, sc=4096 ** -0.5), rnd(100, 14336), rnd(4096, 14336, sc=14336 ** -0.5)
    assert ctx.qkv_project_workspace_bytes(100, 4096) > 0 and ctx.linear_workspace_bytes(100, 14336, 4096) > 0
    outs = [torch.empty((100, n), dtype=torch.bfloat16, device="cuda") for n in (1024, 256, 256, 4096)]

    def call(**kw):
        for o in outs:
            o.fill_(float("nan"))
        ctx.qkv_project(x, w_qkv, *outs[:3], **kw)
        ctx.linear(a, w_down, outs[3], residual=x, **kw)
        return outs
    return call


def _same(a, b):
    return all(torch.equal(s.view(torch.uint8), t.view(torch.uint8)) for s, t in zip(a, b))


def test_products_in_parts_replay_in_a_hip_graph():
    # (the scratch of a captured call is the graph's own: eager calls and other tensors in between do not get it)
    call = _products_in_parts()
    none = torch.empty(0, dtype=torch.uint8, device="cuda")
    whole = [t.clone() for t in call(workspace=none)]
    want = [t.clone() for t in call()]
    assert not _same(want, whole), "the two sums round alike: nothing to tell them apart by"
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        outs = call()
    for rep in range(3):
        other = [torch.full((n << 20,), rep + 1, dtype=torch.uint8, device="cuda") for n in (1, 3, 8, 24)]
        assert _same(call(), want)
        torch.cuda.synchronize()
        graph.replay(); torch.cuda.synchronize()
        assert _same(outs, want), f"replay {rep}"
        assert all(bool((t == rep + 1).all()) for t in other)


def test_products_without_memory_for_their_parts_stay_whole(monkeypatch):
    call = _products_in_parts()
    none = torch.empty(0, dtype=torch.uint8, device="cuda")
    whole = [t.clone() for t in call(workspace=none)]
    torch.cuda.synchronize()
    # a capture that torch does not know of
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)
    assert _same(call(), whole)
    # an allocator that does not say where its memory lies
    def silent():
        raise RuntimeError("no snapshot")
    monkeypatch.setattr(torch.cuda, "memory_snapshot", silent)
    assert _same(call(), whole)
    monkeypatch.undo()
    # no memory
    def refuse(*args, **kw):
        raise torch.cuda.OutOfMemoryError("no memory")
    monkeypatch.setattr(torch, "empty", refuse)
    got = [t.clone() for t in call()]
    monkeypatch.undo()
    assert _same(got, whole)
    assert not _same(call(), whole)


def test_products_while_another_thread_captures():
    # a size that the allocator has no memory for yet, on another stream: neither the call nor the capture may fail
    import threading
    call = _products_in_parts()
    want = [t.clone() for t in call()]
    a = torch.ones(1 << 20, device="cuda")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    got, failed = [], []

    def other():
        try:
            with torch.cuda.stream(stream):
                got.extend(call())
        except Exception as e:                           # (reported by the assertion below)
            failed.append(e)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        a.mul_(2.0)
        t = threading.Thread(target=other)
        t.start(); t.join()
    torch.cuda.synchronize()
    assert not failed, failed
    assert _same(got, want)
    graph.replay(); torch.cuda.synchronize()
    assert bool((a == 2.0).all())
