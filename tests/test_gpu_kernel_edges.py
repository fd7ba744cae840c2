"""Kernels at the sizes where their loops and splits change: edges of tiles, remainders, the smallest and the
largest of a range.  Needs an MI355X (-m gpu)."""
import math

import numpy as np
import pytest
import torch

import workload as W
from oracle import cachecraft_oracle as O
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[1, 2, 63, 64, 65], [255, 256, 257, 511], [1023, 4096], [4097]])
@pytest.mark.parametrize("frac", [0.0, 0.01, 0.37, 1.0])
def test_top_n_around_the_lengths_where_its_loops_change(lens, frac):
    # (a wavefront owns 64-token rounds of a quarter of the chunk; up to 4096 tokens stay in registers)
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("topn", "f32", 2, 1, 64, 1.0e4, lens, [0] * len(lens),
                 [W.RequestSpec(list(range(len(lens))), [frac] * len(lens), 3)], 1.0, seed=13)
    rng = np.random.default_rng(len(lens))
    ties = rng.integers(0, 9, size=w.n_tok) / np.float32(8)                     # few distinct values
    for given in (rng.standard_normal(w.n_tok), ties, np.zeros(w.n_tok), 0.75 + 1e-6 * rng.random(w.n_tok)):
        given = given.astype(np.float32)
        b = DeviceBatch(w)
        b.select_from_scores(torch.from_numpy(given).cuda()); torch.cuda.synchronize()
        for got, sg in zip(H.gpu_selection(w, b.sel_idx.cpu().numpy())[0], H.chunk_segments(w, 0)):
            t0, n = int(sg[W.SEG_TOK]), int(sg[W.SEG_NTOK])
            assert np.array_equal(got, O.top_n(given[t0:t0 + n].astype(np.float64), int(sg[W.SEG_NSEL])))


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("hkv", [1, 3, 8])
def test_scatter_runs_of_every_length_at_every_place(dtype, d, hkv):
    # runs of 1..16 rows that start at every offset of a workgroup's four candidate rows, slots in any order
    # inside a block, rows with a slot outside the pool between them
    import paper_2502_15734_amd as P
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = np.random.default_rng(hkv)
    lengths = [1, 16, 2, 1, 15, 3, 5, 16, 7, 1, 1, 4, 16, 9, 2, 16, 16, 1]
    blocks = rng.permutation(len(lengths) + 3)[: len(lengths)]
    slots, n_blocks = [], len(lengths) + 3
    for i, (b, m) in enumerate(zip(blocks, lengths)):
        slots += [int(b) * 16 + int(s) for s in rng.permutation(16)[:m]]
        if i % 5 == 3:
            slots.append(-1 if i % 2 else n_blocks * 16)
    n = len(slots)
    pos = rng.integers(0, 30000, size=n).astype(np.int32)
    ctx = P.Context(hkv, hkv, d, 5.0e5, P.CC_BF16 if dtype == "bf16" else P.CC_F32)
    g = torch.Generator(device="cuda").manual_seed(5)
    k_new, v_new = (torch.randn(n, hkv, d, device="cuda", generator=g).to(dt) for _ in range(2))
    k_pool = torch.randn(n_blocks, hkv, 16, d, device="cuda", generator=g).to(dt)
    v_pool = torch.randn(n_blocks, hkv, d, 16, device="cuda", generator=g).to(dt)
    want_k, want_v = k_pool.cpu().double().numpy(), v_pool.cpu().double().numpy()
    ang = pos[:, None].astype(np.float64) * 5.0e5 ** (-2.0 * np.arange(d // 2) / d)
    cs, sn = np.cos(ang)[:, None], np.sin(ang)[:, None]
    kn = k_new.cpu().double().numpy()
    x, y = kn[..., : d // 2], kn[..., d // 2:]
    turned = np.concatenate([x * cs - y * sn, y * cs + x * sn], axis=-1)
    for j, s in enumerate(slots):
        if 0 <= s < n_blocks * 16:
            want_k[s // 16, :, s % 16] = turned[j]
            want_v[s // 16, :, :, s % 16] = v_new[j].cpu().double().numpy()
    dev = lambda a: torch.from_numpy(np.asarray(a, dtype=np.int32)).cuda()
    ctx.scatter_kv(k_new, v_new, dev(pos), dev(slots), k_pool, v_pool); torch.cuda.synchronize()
    assert np.array_equal(v_pool.cpu().double().numpy(), want_v)
    got_k = k_pool.cpu().double().numpy()
    # half a unit in the last place of the stored value (bf16: 8 significant bits, so 2^-8 of it; fp32: 2^-24) and
    # the fp32 rotation: a few 2^-24 of |x| + |y|, which stay below 8 here; the hardware sine / cosine of the
    # bf16 form: 1e-6 of them
    tol = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -24
    slack = 8 * (1e-6 if dtype == "bf16" else 4 * 2.0 ** -24)
    worst = float(np.max(np.abs(got_k - want_k) - tol * np.abs(want_k)))
    assert worst <= slack


@pytest.mark.parametrize("dtype,d,hq,hkv", [("f32", 64, 4, 2), ("f32", 128, 3, 1), ("bf16", 64, 6, 2), ("bf16", 128, 3, 1)])
@pytest.mark.parametrize("lens,question", [([15, 16, 17], 1), ([8209, 33], 18)])
def test_fp32_arithmetic_kernels_against_the_scalar_ones(dtype, d, hq, hkv, lens, question):
    # one row more or less than a 16-row tile and a 16-token block; more key blocks (515) than one list window (512)
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("f32k", dtype, hq, hkv, d, 1.0e4, lens, [3] * len(lens),
                 [W.RequestSpec(list(range(len(lens))), [0.003] * len(lens), question)], 1.0, seed=31)
    got = {}
    for impl in (P.CC_IMPL_AUTO, P.CC_IMPL_SCALAR):
        b = DeviceBatch(w, impl=impl, poison=True)
        b.rope_shift(); b.select()
        if impl == P.CC_IMPL_SCALAR:
            sel = got[P.CC_IMPL_AUTO][0]
            b.set_selection(*sel)
        else:
            sel = tuple(t.cpu().numpy()[: w.n_q_tot] for t in (b.sel_idx, b.q_row, b.q_pos, b.slot_map))
        b.sparse_prefill_fused(); torch.cuda.synchronize()
        got[impl] = (sel, b.scores.cpu().double(), b.out.cpu().double(), b.lse.cpu().double())
    a, s = got[P.CC_IMPL_AUTO], got[P.CC_IMPL_SCALAR]
    # both sum n fp32 terms of one sign in different orders: n 2^-24 at the very worst, sqrt(n) 2^-24 in practice
    n_ctx = sum(lens) + question
    rel = lambda x, y: float((x - y).norm() / y.norm())
    bound = 8 * math.sqrt(n_ctx) * 2.0 ** -24 + 1e-6                             # + the exponentials' own error
    assert rel(a[1], s[1]) <= bound
    assert rel(a[2], s[2]) <= bound + (2.0 ** -9 if dtype == "bf16" else 0.0)    # (bf16 output: a rounding may flip)
    assert float((a[3] - s[3]).abs().max()) <= 8 * bound


@pytest.mark.parametrize("n_in", [64, 128, 192, 640])
@pytest.mark.parametrize("op,n_out,rows", [
    ("linear", 64, 65), ("linear", 192, 127), ("linear", 256, 300), ("linear", 4096, 31), ("linear", 4096, 129),
    ("linear", 4096, 513), ("linear", 4096, 1025), ("linear", 8192, 2305), ("linear", 32768, 257),
    ("gated", 96, 33), ("gated", 4096, 64), ("gated", 4096, 449), ("gated", 8192, 1281),
    ("qkv", 6144, 15), ("qkv", 6144, 449), ("qkv", 6144, 2817)])
def test_matrix_products_of_every_tile_shape(op, n_out, rows, n_in):
    # one row and one tile more or less than the shapes of the dispatch (32 x 64 ... 256 x 256 features x tokens, and
    # whole rounds of the largest with the remainder in another launch), contraction lengths of one stage and up
    import paper_2502_15734_amd as P
    g = torch.Generator(device="cuda").manual_seed(rows)
    rnd = lambda *s, sc=1.0: (torch.randn(*s, device="cuda", generator=g) * sc).to(torch.bfloat16)
    ctx = P.Context(32, 8, 128, 5.0e5, P.CC_BF16)
    x, w = rnd(rows, n_in), rnd(n_out * (2 if op == "gated" else 1), n_in, sc=n_in ** -0.5)
    nan = lambda n: torch.full((rows, n), float("nan"), dtype=torch.bfloat16, device="cuda")
    product = x.float() @ w.float().t()
    if op == "qkv":
        got = [nan(n) for n in (4096, 1024, 1024)]
        ctx.qkv_project(x, w, *got)
        got, want = torch.cat(got, dim=1), product
    elif op == "gated":
        got = nan(n_out)
        ctx.gated_linear(x, w[:n_out], w[n_out:], got)
        want = torch.nn.functional.silu(product[:, :n_out]) * product[:, n_out:]
    else:
        got, res = nan(n_out), rnd(rows, n_out)
        ctx.linear(x, w, got, residual=res)
        want = product + res.float()
    torch.cuda.synchronize()
    # half a unit in the last place of bf16, and fp32 sums of n_in products of size n_in^-1/2 in two orders
    assert float(((got.float() - want).abs() - 2.0 ** -8 * want.abs()).max()) <= 8 * n_in * 2.0 ** -24 * 4


@pytest.mark.parametrize("lens,frac,question", [([5], 0.4, 1), ([64], 0.25, 15), ([70, 60], 0.25, 1), ([129, 1, 0, 190], 0.1, 33),
                                                ([300], 0.4, 65), ([2000, 6250, 40], 0.004, 31)])
def test_attention_in_two_key_streams(lens, frac, question):
    # grids of a few workgroups (here: one to three row tiles of one KV head): the even and the odd 64-key tiles are
    # walked apart.  One tile (an odd stream without keys), rows that see only the first tile, an odd count, rows
    # around a 32-row tile, segments that end in either stream or have no tokens, more than 64 tiles per stream.
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("streams", "bf16", 4, 1, 128, 5.0e5, lens, [0] * len(lens),
                 [W.RequestSpec(list(range(len(lens))), [frac] * len(lens), question)], 1.0, seed=47)
    b = DeviceBatch(w, poison=True)
    b.rope_shift(); b.select(); b.gather(); b.sparse_prefill(); torch.cuda.synchronize()
    sel = tuple(t.cpu().numpy()[: w.n_q_tot] for t in (b.sel_idx, b.q_row, b.q_pos, b.slot_map))
    s = DeviceBatch(w, impl=P.CC_IMPL_SCALAR, poison=True)
    s.rope_shift(); s.set_selection(*sel); s.gather(); s.sparse_prefill(); torch.cuda.synchronize()
    n = w.n_q_tot
    out, ref = b.out[:n].double(), s.out[:n].double()
    assert float((out - ref).norm() / ref.norm()) <= H.TOL["bf16"]
    # the rotated query is rounded to bf16 (a relative 2^-9 / sqrt(3) in the mean, per product of variance 1 / 128): a row
    # that sees a single key shows it whole, 2^-9 / sqrt(3) = 1.1e-3; six of these
    assert float((b.lse[:n] - s.lse[:n]).abs().max()) <= 6.8e-3
    # the by-product form walks the same way: the same bits, and the question's masses of the separate kernel
    out1, lse1, m1 = b.out[:n].clone(), b.lse[:n].clone(), s.question_mass().cpu()
    m2 = b.sparse_prefill_mass().cpu()
    assert torch.equal(out1, b.out[:n]) and torch.equal(lse1, b.lse[:n])
    assert torch.isfinite(m2).all() and abs(float(m2.sum()) - question) <= 3e-3 * question
    assert float((m1 - m2).abs().max()) <= 2e-2


@pytest.mark.parametrize("hq", [4, 8])
@pytest.mark.parametrize("lens", [[5, 3], [64, 64], [1, 129], [63, 65, 1, 0, 190], [128, 130], [2000, 6250, 40]])
def test_scores_in_two_key_streams(hq, lens):
    # grids below the wide form's: 64-token workgroups whose even and odd 64-key tiles are walked apart.  A stream without
    # tiles of the chunk itself or with one tile less, chunks around a 32-token column block and a 64-token tile, a
    # segment without tokens, more than 64 tiles per stream.
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("scores2", "bf16", hq, 1, 128, 5.0e5, lens, [7] * len(lens),
                 [W.RequestSpec(list(range(len(lens))), [0.2] * len(lens), 9)], 1.0, seed=53)
    for gain in (1.0, 40.0):
        got = []
        for impl in (P.CC_IMPL_AUTO, P.CC_IMPL_MFMA_NARROW):
            b = DeviceBatch(w, impl=impl, poison=True)
            b.q.mul_(gain)
            b.rope_shift(); b.select(); torch.cuda.synchronize()
            got.append(b.scores.cpu().double())
        # both round the same rotated queries to bf16 (every angle is taken in double precision), so only the order of the
        # fp32 sums differs: sqrt(n) 2^-24 of a sum, four of these (prior and own, two kernels), and the hardware exponential's
        # 1e-6 for logits that are subtracted from a reference or not; larger queries in proportion (their sums leave the safe
        # range and are redone by the narrow kernel).  An angle wrong by 1e-6 turns roundings over: 5e-6 to 2e-5
        assert torch.isfinite(got[0]).all()
        assert float((got[0] - got[1]).abs().max()) <= (4 * math.sqrt(sum(lens)) * 2.0 ** -24 + 1e-6) * gain
        assert float(got[1].max()) > 0.1


@pytest.mark.parametrize("dtype,d,hq,hkv,lens,fracs,cut", [
    # two key streams: 32 rows that see the first 64-key tile only, tiles of both streams behind it
    ("bf16", 128, 4, 1, [64, 70], [0.5, 0.1], 64), ("bf16", 128, 8, 2, [64, 300, 20], [0.5, 0.1, 0.3], 64),
    # fp32 arithmetic: rows in front of and behind `cut` share a 16-row tile, `cut` inside and at the edge of a 16-token block
    ("f32", 64, 4, 2, [40, 30], [0.5, 0.2], 37), ("f32", 128, 3, 1, [21, 300, 20], [0.4, 0.02, 0.3], 16),
    ("bf16", 64, 6, 2, [40, 30], [0.5, 0.2], 37), ("bf16", 128, 3, 1, [700, 5], [0.01, 0.4], 301)])
def test_values_behind_a_rows_position_do_not_reach_it(dtype, d, hq, hkv, lens, fracs, cut):
    # values of every token at position `cut` and later are not finite; rows in front of it must be what they are without
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("behind", dtype, hq, hkv, d, 1.0e4, lens, [2] * len(lens),
                 [W.RequestSpec(list(range(len(lens))), fracs, 5)], 1.0, seed=61)
    b = DeviceBatch(w, poison=True)
    b.rope_shift(); b.select()
    got = []
    for plant in (False, True):
        if plant:
            bad = [float("nan"), float("inf"), -float("inf")]
            pos = 0
            for c, n in enumerate(lens):
                for t in range(max(cut - pos, 0), n):
                    blk = int(w.store_tab[int(w.store_tab_off[c]) + t // 16])
                    b.v_store[blk, :, :, t % 16] = bad[t % 3]
                pos += n
            b.v_new[cut:] = bad[0]
            b.rope_shift()                                       # (the value map points into the store again)
        b.sparse_prefill_fused(); torch.cuda.synchronize()
        n = w.n_q_tot
        front = b.q_pos[:n] < cut
        got.append((b.out[:n][front].clone(), b.lse[:n][front].clone()))
    assert int(front.sum()) > 0 and torch.isfinite(got[0][0]).all()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("dtype,d,hq,hkv", [("f32", 64, 4, 2), ("f32", 128, 3, 1), ("bf16", 64, 6, 2), ("bf16", 128, 3, 1)])
def test_fp32_arithmetic_gives_values_that_are_not_finite_to_the_rows_that_see_them(dtype, d, hq, hkv):
    # single dimensions of single tokens, one or two in a block; rows in front of, at and behind each of them in one tile
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("infs", dtype, hq, hkv, d, 1.0e4, [70, 90], [2, 2], [W.RequestSpec([0, 1], [0.3, 0.2], 20)], 1.0, seed=67)
    bad = [float("nan"), float("inf"), -float("inf")]
    got = []
    for impl in (P.CC_IMPL_AUTO, P.CC_IMPL_SCALAR):
        b = DeviceBatch(w, impl=impl, poison=True)
        for i, (c, t) in enumerate([(0, 9), (0, 33), (0, 34), (1, 0), (1, 15), (1, 88)]):
            b.v_store[int(w.store_tab[int(w.store_tab_off[c]) + t // 16]), :, (11 * i) % d, t % 16] = bad[i % 3]
        b.v_new[163, :, 5 + 16] = bad[1]                          # a token of the question (positions 160 to 179)
        b.rope_shift(); b.select()
        if got:
            b.set_selection(*got[0][0])
        sel = tuple(t.cpu().numpy()[: w.n_q_tot] for t in (b.sel_idx, b.q_row, b.q_pos, b.slot_map))
        b.sparse_prefill_fused(); torch.cuda.synchronize()
        got.append((sel, b.out.cpu().double(), b.lse.cpu()))
    a, s = got[0][1], got[1][1]
    assert not torch.isfinite(s).all() and torch.isfinite(s).any(dim=-1).all()
    for what in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(what(a), what(s))
    ok = torch.isfinite(s)
    # (two orders of fp32 sums over 180 keys, and a rounding of a bf16 output that may flip)
    assert float((a - s)[ok].norm() / s[ok].norm()) <= 8 * math.sqrt(180) * 2.0 ** -24 + 1e-6 + (2.0 ** -9 if dtype == "bf16" else 0.0)
    assert torch.isfinite(got[0][2]).all()


@pytest.mark.parametrize("d,hq,hkv", [(64, 4, 2), (64, 8, 2), (128, 3, 1)])
@pytest.mark.parametrize("lens", [[20, 36], [17, 60, 45], [150, 200, 180]])
def test_fp32_arithmetic_is_no_further_from_64_bits_than_the_scalar_kernels(d, hq, hkv, lens):
    # (both read the same fp32 keys and values; a logit summed in one chain of d additions fails this on the short prompts)
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("err", "f32", hq, hkv, d, 1.0e4, lens, [3] * len(lens),
                 [W.RequestSpec(list(range(len(lens))), [0.2] * len(lens), 20)], 1.0, seed=71)
    err, sel = [], None
    for impl in (P.CC_IMPL_AUTO, P.CC_IMPL_SCALAR):
        b = DeviceBatch(w, impl=impl, cow=False)
        b.rope_shift()
        if sel is None:
            b.select()
            sel = tuple(t.cpu().numpy()[: w.n_q_tot] for t in (b.sel_idx, b.q_row, b.q_pos, b.slot_map))
        else:
            b.set_selection(*sel)
        b.sparse_prefill_fused(); torch.cuda.synchronize()
        k, v = H.request_context_from_pools(w, 0, b.k_req.cpu().double().numpy(), b.v_req.cpu().double().numpy())
        out, _ = O.causal_attention_rows_dense(O.rotate(w.q[sel[1]].astype(np.float64), sel[2], 1.0e4), sel[2], k, v)
        err.append(H.rel_l2(b.out.cpu().numpy(), out))
    assert err[0] <= err[1], err


def test_wide_runs_the_form_of_large_grids_at_every_size():
    # one request alone, asked for the wide kernels, and as one of 32 equal ones whose grid AUTO gives to the same form
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    got = []
    for n, impl in ((1, P.CC_IMPL_MFMA_WIDE), (32, P.CC_IMPL_AUTO)):
        w = W.custom("alone", "bf16", 8, 2, 128, 5.0e5, [300, 290, 210], [4, 4, 4],
                     [W.RequestSpec([0, 1, 2], [0.2, 0.2, 0.2], 30)] * n, 1.0 / math.sqrt(128), seed=83)
        one = w.n_tok // n
        rng = np.random.default_rng(5)
        for t in (w.q, w.k_new, w.v_new):
            t[:] = np.tile(rng.standard_normal((one,) + t.shape[1:]).astype(t.dtype), (n, 1, 1))
        b = DeviceBatch(w, impl=impl, poison=True)
        b.rope_shift(); b.select_from_scores(torch.from_numpy(np.tile(rng.random(one).astype(np.float32), n)).cuda())
        b.sparse_prefill_fused(); torch.cuda.synchronize()
        m = w.n_q_tot // n
        got.append((b.out[:m].clone(), b.lse[:m].clone()))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("impl", ["AUTO", "MFMA_WIDE"])
@pytest.mark.parametrize("low", [(0, 32), (64, 96), (64, 128)])
def test_rows_whose_reference_lies_far_below_later_keys(impl, low):
    # keys with logits around -100 in the first block of the even (or only) or of the odd key stream: its sums leave fp32's
    # range and the rows are redone by the kernel that moves its reference
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("lowref2", "bf16", 8, 2, 128, 5.0e5, [300, 180, 150], [0, 0, 0],
                 [W.RequestSpec([0, 1, 2], [0.25, 0.25, 0.25], 40)], 1.0 / math.sqrt(128), seed=21)
    w.q[:, :, 60:64] = 2.0
    w.q[:, :, 124:128] = 0.0
    blocks = w.store_tab[w.store_tab_off[0]: w.store_tab_off[1]]
    for t in range(*low):
        w.k_store[blocks[t // 16], :, t % 16, 60:64] = -141.0
        w.k_store[blocks[t // 16], :, t % 16, 124:128] = 0.0
    w.k_new[low[0]:low[1], :, 60:64] = -141.0
    w.k_new[low[0]:low[1], :, 124:128] = 0.0
    b = DeviceBatch(w, impl=getattr(P, "CC_IMPL_" + impl), poison=True)
    b.step(); torch.cuda.synchronize()
    ref = O.run_request(w, 0, selected_override=H.gpu_selection(w, b.sel_idx.cpu().numpy())[0])
    assert H.rel_l2(b.out.float().cpu().numpy(), ref.out) <= H.TOL["bf16"]
    # (rows that see nothing but such keys: bf16 keys of magnitude 141, half a unit in the last place of four of them)
    only = (ref.q_pos < low[1]) if low[0] == 0 else np.zeros(len(ref.q_pos), dtype=bool)
    assert (np.abs(b.lse.cpu().numpy() - ref.lse) <= np.where(only[:, None], 0.8, 2e-3)).all()


@pytest.mark.parametrize("hq,hkv,n,lens", [(32, 8, 4, [512] * 3), (64, 8, 4, [100] * 5)])
def test_scores_of_grids_between_the_two_wide_forms_come_from_the_narrow_kernel(hq, hkv, n, lens):
    # more 64-token workgroups than two key streams have a round for, prompts too short to gain from the shorter chain
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("between", "bf16", hq, hkv, 128, 5.0e5, lens, [3] * len(lens),
                 [W.RequestSpec(list(range(len(lens))), [0.1] * len(lens), 20)] * n, 1.0 / math.sqrt(128), seed=89)
    got = []
    for impl in (P.CC_IMPL_AUTO, P.CC_IMPL_MFMA_NARROW):
        b = DeviceBatch(w, impl=impl)
        b.rope_shift(); b.select(); torch.cuda.synchronize()
        got.append(b.scores.cpu())
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("hq,lens,chunks", [
    (4, [40, 1, 63, 65, 0, 128, 200, 31], [[0, 1, 2, 3, 4, 5, 6, 7], [6, 0], [3], [1, 1, 1, 2]]),
    (8, [130, 126, 257, 5], [[0, 1, 2, 3], [3, 3, 3, 0, 2]]),
    (4, [9, 3, 20], [[0, 1, 2] * 30, [2, 1]]),                  # more than 64 segments in a request
    (4, [17, 33], [[0, 1, 0]] * 300),                           # more than 1024 segments
    (4, [17, 20], [[0, 1]] * 2100),                             # more requests than are sorted
])
def test_scores_of_tokens_numbered_through_the_chunks_of_a_request(hq, lens, chunks):
    # a workgroup's 128 (64) tokens begin and end anywhere in a chunk and may lie in many: each column takes its own prior
    # chunks' mass where its own chunk begins
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("through", "bf16", hq, 1, 128, 5.0e5, lens, [7] * len(lens),
                 [W.RequestSpec(c, [0.2] * len(c), 5) for c in chunks], 1.0, seed=97)
    longest = max(sum(lens[i] for i in c) for c in chunks)
    for gain in (1.0, 40.0):
        got = {}
        for impl in ("MFMA_NARROW", "MFMA_WIDE", "AUTO"):
            b = DeviceBatch(w, impl=getattr(P, "CC_IMPL_" + impl), poison=True)
            b.q.mul_(gain)
            b.rope_shift(); b.select(); torch.cuda.synchronize()
            got[impl] = b.scores.cpu().double()
        # (the bound of test_scores_in_two_key_streams: every form takes every angle in double precision)
        bound = (4 * math.sqrt(longest) * 2.0 ** -24 + 1e-6) * gain
        for impl in ("MFMA_WIDE", "AUTO"):
            assert torch.isfinite(got[impl]).all()
            assert float((got[impl] - got["MFMA_NARROW"]).abs().max()) <= bound
    assert float(got["MFMA_NARROW"].max()) > 0.1


@pytest.mark.parametrize("lens", [[7, 15], [16, 17], [33, 16, 15, 1], [64, 49, 80], [70, 130, 3]])
def test_scores_of_the_wide_form_around_16_tokens_and_16_keys(lens):
    # the form of large grids multiplies 16 tokens by 16 keys: last tokens, chunk boundaries and causal edges one short of
    # such a block, on it and one behind it
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("halves", "bf16", 4, 1, 128, 5.0e5, lens, [7] * len(lens),
                 [W.RequestSpec(list(range(len(lens))), [0.2] * len(lens), 9)], 1.0, seed=29)
    for gain in (1.0, 40.0):
        got = []
        for impl in (P.CC_IMPL_MFMA_WIDE, P.CC_IMPL_MFMA_NARROW):
            b = DeviceBatch(w, impl=impl, poison=True)
            b.q.mul_(gain)
            b.rope_shift(); b.select(); torch.cuda.synchronize()
            got.append(b.scores.cpu().double())
        # (the bound of test_scores_in_two_key_streams)
        assert torch.isfinite(got[0]).all()
        assert float((got[0] - got[1]).abs().max()) <= (4 * math.sqrt(sum(lens)) * 2.0 ** -24 + 1e-6) * gain
        assert float(got[1].max()) > 0.1


@pytest.mark.parametrize("lens,n_requests,columns", [([16, 17, 1], 24, 32), ([33, 16, 15, 1], 24, 32), ([64, 49, 80], 24, 32), ([70, 130, 3], 24, 32), ([5, 31, 33], 24, 32),
                                                     ([590, 589, 590, 600, 590, 577, 590, 590], 1, 32), ([700, 689, 702, 700, 711], 2, 16)])
def test_scores_of_short_and_of_long_calls_on_large_grids(lens, n_requests, columns):
    # short calls multiply 32 columns, long ones 16 (as the forced wide kernel always does): last tokens, chunk boundaries and causal edges around 16 and 32
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("columns", "bf16", 64, 8, 128, 5.0e5, lens, [7] * len(lens),
                 [W.RequestSpec(list(range(len(lens))), [0.2] * len(lens), 9) for _ in range(n_requests)], 1.0, seed=31)
    for gain in (1.0, 40.0):
        got = {}
        for impl in ("AUTO", "MFMA_WIDE", "MFMA_NARROW"):
            b = DeviceBatch(w, impl=getattr(P, "CC_IMPL_" + impl), poison=True)
            b.q.mul_(gain)
            b.rope_shift(); b.select(); torch.cuda.synchronize()
            got[impl] = b.scores.cpu().double()
        # (the bound of test_scores_in_two_key_streams; the forms add in different orders, so their bits tell which one ran, unless the second
        # pass has redone what left the safe range)
        assert torch.isfinite(got["AUTO"]).all()
        assert float((got["AUTO"] - got["MFMA_NARROW"]).abs().max()) <= (4 * math.sqrt(sum(lens)) * 2.0 ** -24 + 1e-6) * gain
        if gain == 1.0:
            assert torch.equal(got["AUTO"], got["MFMA_WIDE"]) == (columns == 16) and not torch.equal(got["AUTO"], got["MFMA_NARROW"])
        assert float(got["MFMA_NARROW"].max()) > 0.1


@pytest.mark.parametrize("n_requests", [65536, 65537])
def test_scores_behind_many_empty_requests(n_requests):
    # a list entry has 32 bits for request and row tile: 16 for the one and 16 for the other, 17 and 15
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    lens = [70, 129, 200]
    w = W.custom("empty", "bf16", 8, 1, 128, 5.0e5, lens, [7] * 3, [W.RequestSpec([0, 1, 2], [0.2] * 3, 5)], 1.0, seed=98)
    got = {}
    for impl in ("MFMA_NARROW", "AUTO"):
        b = DeviceBatch(w, impl=getattr(P, "CC_IMPL_" + impl), poison=True)
        b.rope_shift()
        if impl == "AUTO":
            seg = b.segments.cpu().numpy().copy()
            assert (seg[:, 0] == 0).all()
            seg[:, 0] = n_requests - 1
            off = np.zeros(n_requests + 1, dtype=np.int32)
            off[n_requests] = len(seg)
            b.segments, b.req_seg_off, b.n_requests = torch.from_numpy(seg).cuda(), torch.from_numpy(off).cuda(), n_requests
        b.select(); torch.cuda.synchronize()
        got[impl] = b.scores.cpu().double()
    # (the bound of test_scores_in_two_key_streams)
    assert torch.isfinite(got["AUTO"]).all() and float(got["MFMA_NARROW"].max()) > 0.1
    assert float((got["AUTO"] - got["MFMA_NARROW"]).abs().max()) <= 4 * math.sqrt(sum(lens)) * 2.0 ** -24 + 1e-6


@pytest.mark.parametrize("hq,hkv,lens,reqs", [
    (8, 2, [200, 90, 330], [([0, 1, 2], 0.3, 20), ([2, 2], 0.02, 1), ([1], 1.0, 64), ([0], 0.0, 3)]),
    (8, 1, [700, 64], [([0, 0, 0, 0], 0.11, 70), ([1, 0], 0.5, 9)] * 5),      # rows far apart: the halves see other tiles
    (4, 1, [17, 20], [([0, 1], 0.2, 2)] * 2100),                               # more requests than are sorted, no list
    (4, 1, [40], [([0], 1.0, 2)] * 3),                                         # (nearly) every token is a row
])                                                                             # (small grids have no list: test_attention_from_a_sorted_list)
def test_attention_of_several_requests_from_the_list_of_workgroups(hq, hkv, lens, reqs):
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("listed", "bf16", hq, hkv, 128, 5.0e5, lens, [3] * len(lens),
                 [W.RequestSpec(c, [f] * len(c), u) for c, f, u in reqs], 1.0 / math.sqrt(128), seed=101)
    scores = torch.from_numpy(np.random.default_rng(5).random(w.n_tok).astype(np.float32)).cuda()
    got = {}
    for impl in ("MFMA_NARROW", "MFMA_WIDE", "AUTO"):
        b = DeviceBatch(w, impl=getattr(P, "CC_IMPL_" + impl), poison=True)
        b.rope_shift(); b.select_from_scores(scores); b.sparse_prefill_fused(); torch.cuda.synchronize()
        n = w.n_q_tot
        got[impl] = b.out[:n].double().cpu().numpy(), b.lse[:n].double().cpu()
    for impl in ("MFMA_WIDE", "AUTO"):
        # both round P and the output to bf16: 2^-9 each, twice; the sums of up to n keys: sqrt(n) 2^-24, the hardware's
        # exponential and logarithm 1e-6 each, twice
        assert np.isfinite(got[impl][0]).all()
        assert H.rel_l2(got[impl][0], got["MFMA_NARROW"][0]) <= 4 * 2.0 ** -9
        assert float((got[impl][1] - got["MFMA_NARROW"][1]).abs().max()) <= 2 * (60 * 2.0 ** -24 + 2e-6) * 8
    # the by-product form takes the same rows in the same workgroups: the same bits
    out1, lse1 = b.out[:n].clone(), b.lse[:n].clone()
    b.rope_shift(); b.select_from_scores(scores); mass = b.sparse_prefill_mass(fused=True).cpu()
    assert torch.equal(out1, b.out[:n]) and torch.equal(lse1, b.lse[:n])
    sums = torch.zeros(w.n_requests).index_add_(0, torch.from_numpy(w.segments[:, W.SEG_REQ].astype(np.int64)), mass)
    assert float((sums - torch.tensor([float(u) for _, _, u in reqs])).abs().max()) <= 3e-3 * max(u for _, _, u in reqs)


@pytest.mark.parametrize("hq,hkv,lens,fracs,question", [(4, 1, [3, 1], [1.0, 1.0], 1), (8, 2, [70, 33, 16], [0.3, 1.0, 0.1], 5),
                                                        (24, 3, [130], [0.5], 2), (8, 1, [40, 300], [1.0, 0.2], 17)])
def test_weight_a_row_keeps_on_itself(hq, hkv, lens, fracs, question):
    # rows of four heads at a time, a wavefront per row, four rows per workgroup (remainders 1, 2, 3); groups of 4 and 8 heads
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("self", "bf16", hq, hkv, 128, 5.0e5, lens, [5] * len(lens),
                 [W.RequestSpec(list(range(len(lens))), fracs, question)], 1.0 / math.sqrt(128), seed=103)
    b = DeviceBatch(w, poison=True)
    b.rope_shift(); b.select_from_scores(torch.from_numpy(np.random.default_rng(9).random(w.n_tok).astype(np.float32)).cuda())
    b.gather(); b.sparse_prefill()
    _, self_mass, _ = b.chunk_attention()
    torch.cuda.synchronize()
    # own weights in double precision from what the call itself read: the rows' queries, the fixed pages, its log-sum-exp
    n, k_pool = w.n_q_tot, b.k_req.double().cpu().numpy()
    pos, slot = b.q_pos[:n].cpu().numpy(), b.slot_map[:n].cpu().numpy()
    ang = pos[:, None] * (5.0e5 ** (-2.0 * np.arange(64) / 128))[None]
    c, s = np.cos(ang)[:, None], np.sin(ang)[:, None]
    x, y = np.split(b.q[b.q_row[:n].long()].double().cpu().numpy(), 2, axis=2)
    k = k_pool[slot // 16, :, slot % 16].repeat(hq // hkv, axis=1)
    logit = (np.concatenate([x * c - y * s, y * c + x * s], axis=2) * k).sum(axis=2) / math.sqrt(128)
    own = np.exp(logit - b.lse[:n].double().cpu().numpy()).mean(axis=1)
    ref = np.array([own[(pos >= g[W.SEG_START]) & (pos < g[W.SEG_START] + g[W.SEG_NTOK])].sum() for g in w.segments])
    # fp32: 128 products and the sum over up to n rows and hq heads, the angle's 1e-6, the exponential's 1e-6
    assert np.abs(self_mass.cpu().numpy() - ref).max() <= 1e-5 * max(1.0, ref.max())


@pytest.mark.parametrize("n", [1, 1023, 1025, 2047, 2050])
@pytest.mark.parametrize("dense", [False, True])
def test_scatter_with_one_two_and_four_rows_per_workgroup(n, dense):
    import paper_2502_15734_amd as P
    ctx = P.Context(8, 2, 128, 5.0e5, P.CC_BF16)
    rng = np.random.default_rng(n)
    tok = n if dense else 5 * n
    nb = (tok + 15) // 16 + 3
    idx = np.arange(n) if dense else np.sort(rng.choice(tok, n, replace=False))
    blocks = rng.permutation(nb)
    slot = torch.tensor((blocks[idx // 16] * 16 + idx % 16).astype(np.int32), device="cuda")
    pos = torch.tensor((idx + 7).astype(np.int32), device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(n)
    rnd = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    k_new, v_new, k_pool, v_pool = rnd(n, 2, 128), rnd(n, 2, 128), rnd(nb, 2, 16, 128), rnd(nb, 2, 128, 16)
    k_ref, v_ref = k_pool.double(), v_pool.clone()
    ang = pos.double()[:, None] * (5.0e5 ** (-2.0 * torch.arange(64, dtype=torch.float64, device="cuda") / 128))[None]
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    x, y = k_new.double().split(64, dim=2)
    b, o = slot.long() // 16, slot.long() % 16
    k_ref[b, :, o] = torch.cat([x * c - y * s, y * c + x * s], dim=2)
    v_ref[b, :, :, o] = v_new
    ctx.scatter_kv(k_new, v_new, pos, slot, k_pool, v_pool)
    torch.cuda.synchronize()
    assert torch.equal(v_pool, v_ref)                         # (values are copied; everything else stays)
    # one rounding to bf16 (2^-9 of a value of up to 6) and angles good to 1e-6
    assert float((k_pool.double() - k_ref).abs().max()) <= 2.0 ** -8 * 8


@pytest.mark.parametrize("hidden", [2040, 2048, 2056, 8192, 8200])
def test_rms_norm_where_rows_change_from_wavefronts_to_workgroups(hidden):
    import paper_2502_15734_amd as P
    ctx = P.Context(8, 2, 128, 5.0e5, P.CC_BF16)
    gen = torch.Generator(device="cuda").manual_seed(hidden)
    for n in (1, 5):
        x = torch.empty((n, hidden), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
        g = torch.empty(hidden, dtype=torch.bfloat16, device="cuda").normal_(1.0, 0.1, generator=gen)
        ref = x.double() / (x.double().pow(2).mean(dim=1, keepdim=True) + 1e-5).sqrt() * g.double()
        y = torch.empty_like(x)
        ctx.rms_norm(x, g, 1e-5, y)
        ctx.rms_norm(x, g, 1e-5, x)                           # (in place)
        torch.cuda.synchronize()
        assert torch.equal(x, y)
        # the rounding to bf16, and 1e-6 of the scale
        assert ((y.double() - ref).abs() <= ref.abs() * (2.0 ** -8 + 2e-6)).all()


@pytest.mark.parametrize("pieces", [255, 256, 257, 320, 511, 512, 513, 768, 1000, 1023, 1024])
def test_rms_norm_sums_a_row_in_one_order_whatever_its_length(pieces):
    # 16-byte pieces of a row.  The same row with zeros behind it, 16 or 64 times as long, is summed by a wavefront alone: its sum of
    # squares has to have the same bits (bf16: the squares are exact in fp32, so only the order decides), and with eps = 0
    # its scale is then 4 or 8 times the short row's, exactly
    import paper_2502_15734_amd as P
    ctx = P.Context(8, 2, 128, 5.0e5, P.CC_BF16)
    hidden, n, times = 8 * pieces, 96, 64 if pieces < 256 else 16
    gen = torch.Generator(device="cuda").manual_seed(pieces)
    x = torch.zeros((n, times * hidden), dtype=torch.bfloat16, device="cuda")
    x[:, :hidden] = torch.empty((n, hidden), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    g = torch.empty(times * hidden, dtype=torch.bfloat16, device="cuda").normal_(1.0, 0.1, generator=gen)
    long, short = torch.empty_like(x), torch.empty((n, hidden), dtype=torch.bfloat16, device="cuda")
    ctx.rms_norm(x, g, 0.0, long)
    ctx.rms_norm(x[:, :hidden].contiguous(), g[:hidden].contiguous(), 0.0, short)
    torch.cuda.synchronize()
    assert torch.equal(long[:, :hidden].float(), short.float() * math.sqrt(times))
    assert float(short.float().pow(2).mean()) > 0.5


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("pieces", [1025, 1087, 1088, 2048, 2050])
def test_rms_norm_of_rows_whose_end_is_read_twice(dtype, pieces):
    import paper_2502_15734_amd as P
    bf = dtype == "bf16"
    torch_dtype, hidden = (torch.bfloat16, 8 * pieces) if bf else (torch.float32, 4 * pieces)
    ctx = P.Context(8, 2, 128, 5.0e5, P.CC_BF16 if bf else P.CC_F32)
    gen = torch.Generator(device="cuda").manual_seed(pieces)
    x = torch.empty((5, hidden), device="cuda").normal_(generator=gen).to(torch_dtype)
    g = torch.empty(hidden, device="cuda").normal_(1.0, 0.1, generator=gen).to(torch_dtype)
    ref = x.double() / (x.double().pow(2).mean(dim=1, keepdim=True) + 1e-5).sqrt() * g.double()
    y = torch.empty_like(x)
    ctx.rms_norm(x, g, 1e-5, y)
    ctx.rms_norm(x, g, 1e-5, x)                               # (in place)
    torch.cuda.synchronize()
    assert torch.equal(x, y)
    # the rounding of the result (two of fp32), and of the scale's sum: up to 260 terms a lane and six steps, rsqrt 1e-7 each way
    assert ((y.double() - ref).abs() <= ref.abs() * ((2.0 ** -8 if bf else 2.0 ** -22) + 2e-6)).all()


def plan_list_of(ws, at, n_tok, n_segs, n_requests):
    """The list of workgroups that a call left in the tile plan at byte `at` of its workspace, as (request, row tile) pairs;
    None if the workspace, filled with 0x7f before the call, holds no list."""
    up, max_tiles = lambda n: -(-n // 256) * 256, n_tok // 64 + n_segs + 1
    first = at + up(4 * (2 * n_segs + 1)) + up(32 * n_segs)
    work = ws[first: first + 32 * max_tiles].cpu().numpy().view(np.int32).reshape(-1, 8)[:, 7]
    if work[-1] == 0x7f7f7f7f:
        return None
    bits = min(31, 32 - (n_requests - 1).bit_length())              # (what the requests leave of an entry names the row tile)
    e = work[: int(work[-1])].view(np.uint32).astype(np.int64)
    return list(zip((e >> bits).tolist(), (e & (1 << bits) - 1).tolist()))


@pytest.mark.parametrize("n_requests", [512, 513])
def test_attention_lists_the_workgroups_of_as_many_requests_as_it_sorts(n_requests):
    # more requests: a list would have gaps, and the grid of (row tiles) x (requests) runs
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    reqs = [([0, 1], 0.2, 2), ([2, 0], 1.0, 5), ([1], 0.0, 1), ([2, 1, 0], 0.5, 33)]
    reqs = [reqs[i % 4] for i in range(n_requests)]
    w = W.custom("many", "bf16", 4, 1, 128, 5.0e5, [17, 20, 130], [3] * 3,
                 [W.RequestSpec(c, [f] * len(c), u) for c, f, u in reqs], 1.0 / math.sqrt(128), seed=107)
    scores = torch.from_numpy(np.random.default_rng(5).random(w.n_tok).astype(np.float32)).cuda()
    got = {}
    for impl in ("MFMA_NARROW", "AUTO"):
        b = DeviceBatch(w, impl=getattr(P, "CC_IMPL_" + impl), poison=True)
        b.ws_prefill.fill_(0x7f)
        b.rope_shift(); b.select_from_scores(scores); b.sparse_prefill_fused(); torch.cuda.synchronize()
        got[impl] = b.out[:w.n_q_tot].double().cpu().numpy()
    entries = plan_list_of(b.ws_prefill, 0, w.n_tok, len(w.segments), n_requests)
    if n_requests == 512:
        assert sorted(entries) == [(r, k) for r in range(512) for k in range(-(-int(w.cu_q[r + 1] - w.cu_q[r]) // 64))]
    else:
        assert entries is None
    # (the bound of test_attention_of_several_requests_from_the_list_of_workgroups)
    assert np.isfinite(got["AUTO"]).all() and H.rel_l2(got["AUTO"], got["MFMA_NARROW"]) <= 4 * 2.0 ** -9


@pytest.mark.parametrize("requests", [2, 400])
def test_scores_from_a_list_make_no_order_of_segments(requests):
    # (one launch for the whole plan; several beyond 1024 segments)
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("order", "bf16", 4, 1, 128, 5.0e5, [17, 33], [7] * 2, [W.RequestSpec([0, 1, 0], [0.2] * 3, 5)] * requests, 1.0, seed=109)
    n_segs, up = len(w.segments), lambda n: -(-n // 256) * 256
    got = {}
    for impl in ("MFMA_NARROW", "MFMA_WIDE"):
        b = DeviceBatch(w, impl=getattr(P, "CC_IMPL_" + impl), poison=True)
        b.ws_select.fill_(0x7f)
        b.rope_shift(); b.select(); torch.cuda.synchronize()
        at = up(w.n_tok * 4 * 4) + up(w.n_tok * 4) + 4 * (n_segs + 1)              # behind masses, keys and tile offsets
        got[impl] = b.ws_select[at: at + 4 * n_segs].cpu().numpy().view(np.int32), b.scores.cpu().double()
    assert (np.sort(got["MFMA_NARROW"][0]) == np.arange(n_segs)).all() and (got["MFMA_WIDE"][0] == 0x7f7f7f7f).all()
    # (the bound of test_scores_in_two_key_streams)
    assert float((got["MFMA_WIDE"][1] - got["MFMA_NARROW"][1]).abs().max()) <= 4 * math.sqrt(72) * 2.0 ** -24 + 1e-6


def assert_scores_agree(got, ref, hq):
    """Scores of two forms over batches of many tokens (poisoned: a token whose mass nobody wrote would have 3e38)."""
    # Among 1e7 query elements a few are rounded to bf16 the other way (the two forms contract the rotation's products differently):
    # one such moves a logit by up to 2^-8 |q| |k| / sqrt(128), 5e-3 for |q| = |k| = 4, with a random sign per key; over the 17 or more keys
    # of a token and with the slope m (1 - m) <= 1/4 of a mass that is 5e-3 / 4 / 4 of one head's.  Most tokens have none: the sums alone.
    d = (got - ref).abs()
    assert float(d.max()) <= 2.0 ** -8 * 16 / math.sqrt(128) / 16 / hq
    assert float(d.pow(2).mean().sqrt()) <= 1e-6


MIXED = [[0, 1], [2, 0, 2, 1], [3], [1, 3, 0], [2, 2, 2], [3, 3]]


@pytest.mark.parametrize("n_requests,kinds,long", [
    (512, MIXED, 0), (513, MIXED, 0), (769, MIXED, 0),
    (1201, MIXED, 150),                                         # one request of many chunks
    (600, [[0, 2], [], []], 0),                                 # up to 1024 segments: the whole plan is one launch
])
def test_scores_of_as_many_requests_as_are_sorted_and_more(n_requests, kinds, long):
    # every row tile of every request once and nothing else, whatever lies between them (empty chunks and requests without a scored token too)
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    kinds = [kinds[i % len(kinds)] if i != 7 else kinds[7 % len(kinds)] + [0] * long for i in range(n_requests)]
    w = W.custom("sorted", "bf16", 4, 1, 128, 5.0e5, [17, 65, 200, 0], [7] * 4, [W.RequestSpec(k, [0.2] * len(k), 5) for k in kinds], 1.0, seed=113)
    up, seg = lambda n: -(-n // 256) * 256, w.segments
    got = {}
    for impl in ("MFMA_NARROW", "MFMA_WIDE"):
        b = DeviceBatch(w, impl=getattr(P, "CC_IMPL_" + impl), poison=True)
        b.ws_select.fill_(0x7f)
        b.rope_shift(); b.select(); torch.cuda.synchronize()
        got[impl] = b.scores.cpu().double()
    scored = np.zeros(n_requests, dtype=np.int64)
    np.add.at(scored, seg[:, W.SEG_REQ], np.where((seg[:, W.SEG_KIND] == W.KIND_CHUNK) & (seg[:, W.SEG_START] > 0), seg[:, W.SEG_NTOK], 0))
    entries = plan_list_of(b.ws_select, up(w.n_tok * 4 * 4) + up(w.n_tok * 4), w.n_tok, len(seg), n_requests)
    assert sorted(entries) == [(r, k) for r in range(n_requests) for k in range(-(-int(scored[r]) // 128))]
    assert_scores_agree(got["MFMA_WIDE"], got["MFMA_NARROW"], 4)


@pytest.mark.parametrize("hq,hkv,n,lens,chunks,listed", [
    (64, 8, 24, [64, 30], 2, False), (64, 8, 24, [65, 30], 2, True), (64, 8, 24, [64, 30], 3, True),
    (32, 8, 341, [17, 64], 2, False), (32, 8, 342, [17, 64], 2, False),      # (1024 segments in one launch of the plan)
    (16, 2, 341, [17, 64], 2, False), (16, 2, 342, [17, 64], 2, True),
])
def test_scores_of_single_chunks_that_fit_a_narrow_workgroup(hq, hkv, n, lens, chunks, listed):
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("single", "bf16", hq, hkv, 128, 5.0e5, lens, [7] * 2,
                 [W.RequestSpec([(i + j) % 2 for j in range(chunks)], [0.2] * chunks, 9) for i in range(n)], 1.0 / math.sqrt(128), seed=131)
    up, got = lambda k: -(-k // 256) * 256, []
    for impl in (P.CC_IMPL_MFMA_NARROW, P.CC_IMPL_AUTO):
        b = DeviceBatch(w, impl=impl, poison=True)
        b.ws_select.fill_(0x7f)
        b.rope_shift(); b.select(); torch.cuda.synchronize()
        got.append(b.scores.cpu().double())
    entries = plan_list_of(b.ws_select, up(w.n_tok * hq * 4) + up(w.n_tok * 4), w.n_tok, len(w.segments), n)
    assert (entries is not None) == listed
    assert listed or torch.equal(got[0], got[1])
    assert_scores_agree(got[1], got[0], hq)


@pytest.mark.parametrize("n_requests,chunk", [(2100, 500), (525, 2000), (420, 2500)])
def test_scores_of_more_tokens_than_16_bits_of_row_tiles(n_requests, chunk):
    # 4.2 M tokens in one call (four chunks a request): more than 65536 row tiles of 64, though no request has more than 160
    import paper_2502_15734_amd as P
    n_seg, n_tok, up = 4 * n_requests, 4 * n_requests * chunk, lambda n: -(-n // 256) * 256
    assert n_tok > 64 * 65536
    hq, pages = 4, -(-chunk // 16)
    ctx = P.Context(hq, 1, 128, 5.0e5, P.CC_BF16)
    gen = torch.Generator(device="cuda").manual_seed(127)
    rnd = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.0 / math.sqrt(128), generator=gen)
    q, k = rnd(n_tok, hq, 128), rnd(4 * pages, 1, 16, 128)                      # (all requests have the same keys)
    seg, i = np.zeros((n_seg, 8), dtype=np.int32), np.arange(n_seg)
    seg[:, W.SEG_REQ], seg[:, W.SEG_START], seg[:, W.SEG_NTOK] = i // 4, i % 4 * chunk, chunk
    seg[:, W.SEG_TAB], seg[:, W.SEG_NSEL], seg[:, W.SEG_TOK], seg[:, W.SEG_SEL] = i % 4 * pages, 1, i * chunk, i
    ints = lambda v: torch.from_numpy(np.ascontiguousarray(v, dtype=np.int32)).cuda()
    lists = [torch.zeros(n_seg, dtype=torch.int32, device="cuda") for _ in range(4)]
    tab, segs, off = ints(np.arange(4 * pages)), ints(seg), ints(4 * np.arange(n_requests + 1))
    got = []
    for impl in (P.CC_IMPL_MFMA_NARROW, P.CC_IMPL_AUTO):
        ctx.set_impl(impl)
        ws = torch.full((ctx.select_workspace_bytes(n_tok, n_seg),), 0x7f, dtype=torch.uint8, device="cuda")      # (masses of 3e38)
        scores = torch.zeros(n_tok, dtype=torch.float32, device="cuda")
        ctx.select(q, k, tab, segs, off, n_requests, chunk, *lists, scores, ws)
        torch.cuda.synchronize()
        got.append(scores)
    entries = plan_list_of(ws, up(n_tok * hq * 4) + up(n_tok * 4), n_tok, n_seg, n_requests)
    assert entries is not None and sorted(entries) == [(r, t) for r in range(n_requests) for t in range(-(-3 * chunk // 128))]
    assert_scores_agree(got[1].double(), got[0].double(), hq)
    assert float(got[0].max()) > 0.1


@pytest.mark.parametrize("question,listed", [(2, True), (3, False)])
def test_attention_lists_as_many_row_tiles_as_it_sorts(question, listed):
    # 512 requests of 192 and 193 rows: 2048 and 2056 row tiles by the launcher's bound
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("tiles", "bf16", 4, 1, 128, 5.0e5, [190], [3], [W.RequestSpec([0], [1.0], question)] * 512, 1.0 / math.sqrt(128), seed=137)
    scores, got = torch.zeros(w.n_tok, device="cuda"), []
    for impl in (P.CC_IMPL_MFMA_NARROW, P.CC_IMPL_AUTO):
        b = DeviceBatch(w, impl=impl, poison=True)
        b.ws_prefill.fill_(0x7f)
        b.rope_shift(); b.select_from_scores(scores); b.sparse_prefill_fused(); torch.cuda.synchronize()
        got.append(b.out[:w.n_q_tot].double().cpu().numpy())
    entries = plan_list_of(b.ws_prefill, 0, w.n_tok, len(w.segments), 512)
    assert (entries is not None) == listed
    assert not listed or sorted(entries) == [(r, k) for r in range(512) for k in range(3)]
    # (the bound of test_attention_of_several_requests_from_the_list_of_workgroups)
    assert np.isfinite(got[1]).all() and H.rel_l2(got[1], got[0]) <= 4 * 2.0 ** -9


@pytest.mark.parametrize("hq,hkv,n,lens,chunks,rows", [
    (32, 8, 3, [17, 58], 40, 0), (32, 8, 6, [17, 58], 40, 128),            # 264, 576 workgroups of 128 tokens
    (16, 2, 6, [17, 58], 40, 0), (16, 2, 8, [17, 58], 40, 128),            # 288, 384
    (16, 2, 12, [17, 20], 20, 64),                                         # as many chunks, few tokens
])
def test_score_kernels_are_chosen_by_the_workgroups_there_are(hq, hkv, n, lens, chunks, rows):
    # and not by the longest chunk times the number of chunks
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("grid", "bf16", hq, hkv, 128, 5.0e5, lens, [7] * 2,
                 [W.RequestSpec([j % 2 for j in range(chunks)], [0.2] * chunks, 9)] * n, 1.0 / math.sqrt(128), seed=139)
    up, got = lambda k: -(-k // 256) * 256, []
    for impl in (P.CC_IMPL_MFMA_NARROW, P.CC_IMPL_AUTO):
        b = DeviceBatch(w, impl=impl, poison=True)
        b.ws_select.fill_(0x7f)
        b.rope_shift(); b.select(); torch.cuda.synchronize()
        got.append(b.scores.cpu().double())
    entries = plan_list_of(b.ws_select, up(w.n_tok * hq * 4) + up(w.n_tok * 4), w.n_tok, len(w.segments), n)
    scored = sum(lens[j % 2] for j in range(1, chunks))
    if rows == 0:
        assert entries is None and torch.equal(got[0], got[1])
    else:
        assert sorted(entries) == [(r, k) for r in range(n) for k in range(-(-scored // rows))]
    assert_scores_agree(got[1], got[0], hq)


@pytest.mark.parametrize("hq,hkv,lens,reqs,listed", [
    # 64, 65, 63 and many rows, none of a chunk, most of the row tiles in two requests
    (32, 8, [60, 700, 3, 200], [([0], 1.0, 4), ([0], 1.0, 5), ([0], 1.0, 3), ([1, 1, 2], 1.0, 70), ([3, 1], 0.0, 1), ([1, 3, 1], 0.4, 64)] * 7, "sorted"),
    (16, 2, [1500, 40], [([0] * 6, 0.9, 9)] + [([1], 0.5, 2)] * 60, "sorted"),                     # short tiles of very uneven requests
    (8, 1, [129, 30], [([0, 1, 0], 0.7, 33), ([1, 1], 1.0, 1)] * 90, "sorted"),                   # many requests of few tiles
    (4, 1, [60], [([0], 1.0, 4)] * 200, ""), (4, 1, [60], [([0], 1.0, 4)] * 201, "at once"),  # 400 workgroups by the launcher's bound, 402
    (4, 1, [1000, 50], [([0] * 33, 0.8, 40), ([1, 1], 1.0, 3), ([1], 0.2, 64)], "sorted"),    # a prompt beyond 512 x 64 tokens: two key tiles per step of the sorting
])
def test_attention_from_a_sorted_list(hq, hkv, lens, reqs, listed):
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("sorted", "bf16", hq, hkv, 128, 5.0e5, lens, [3] * len(lens),
                 [W.RequestSpec(c, [f] * len(c), u) for c, f, u in reqs], 1.0 / math.sqrt(128), seed=149)
    rows, heads, n_requests = np.diff(w.cu_q), hq // 4, w.n_requests
    tiles = int((-(-rows // 64)).sum())
    assert 2 <= n_requests <= 512 and (256 // heads < tiles <= 2048) == (listed == "sorted")      # (what starts at once is not sorted)
    scores, got = torch.from_numpy(np.random.default_rng(5).random(w.n_tok).astype(np.float32)).cuda(), {}
    for impl in ("MFMA_NARROW", "AUTO"):
        b = DeviceBatch(w, impl=getattr(P, "CC_IMPL_" + impl), poison=True)
        b.ws_prefill.fill_(0x7f)
        b.out.fill_(float("nan"))
        b.rope_shift(); b.select_from_scores(scores); b.sparse_prefill_fused(); torch.cuda.synchronize()
        n = w.n_q_tot
        got[impl] = b.out[:n].double().cpu().numpy(), b.lse[:n].double().cpu()
    entries = plan_list_of(b.ws_prefill, 0, w.n_tok, len(w.segments), n_requests)
    assert (entries is not None) == (listed != "")
    if listed:
        assert sorted(entries) == [(r, k) for r in range(n_requests) for k in range(-(-int(rows[r]) // 64))]
    # (the bounds of test_attention_of_several_requests_from_the_list_of_workgroups; sums of up to n keys)
    assert np.isfinite(got["AUTO"][0]).all() and H.rel_l2(got["AUTO"][0], got["MFMA_NARROW"][0]) <= 4 * 2.0 ** -9
    longest = max(sum(lens[i] for i in c) + u for c, _, u in reqs)
    assert float((got["AUTO"][1] - got["MFMA_NARROW"][1]).abs().max()) <= 2 * (max(60, math.sqrt(longest)) * 2.0 ** -24 + 2e-6) * 8


@pytest.mark.parametrize("impl,hq,hkv,lens,chunks", [
    ("MFMA_WIDE", 32, 8, [300, 40, 129, 17], [[0, 1, 2], [1, 1], [0, 0, 0, 3], [2], [3, 2, 0]] * 7),       # 128 tokens a workgroup
    ("MFMA_WIDE", 64, 8, [900, 20], [[0, 0, 0]] + [[1, 1]] * 40),
    ("AUTO", 4, 1, [700, 33, 250], [[0] * 9, [1, 1, 1], [2, 0, 0, 2, 0]] * 2 + [[1, 2]]),                  # 64 tokens
    ("AUTO", 4, 1, [1000, 50], [[0] * 33, [1, 1], [1, 1, 1]]),                                             # ... a prompt beyond 512 x 64 tokens
    ("MFMA_WIDE", 8, 1, [1000, 50], [[0] * 34, [1, 1], [1, 1, 1]]),
])
def test_scores_from_a_sorted_list(impl, hq, hkv, lens, chunks):
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("sorted", "bf16", hq, hkv, 128, 5.0e5, lens, [7] * len(lens), [W.RequestSpec(c, [0.2] * len(c), 5) for c in chunks], 1.0, seed=151)
    rows = 128 if impl == "MFMA_WIDE" else 64
    tiles = [-(-sum(lens[i] for i in c[1:]) // rows) for c in chunks]
    assert (512 if rows == 128 else 256) // (hq // 4) < sum(tiles) <= 2048        # (more than run at a time: sorted)
    up, got = lambda k: -(-k // 256) * 256, []
    for form in ("MFMA_NARROW", impl):
        b = DeviceBatch(w, impl=getattr(P, "CC_IMPL_" + form), poison=True)
        b.ws_select.fill_(0x7f)                                                    # (masses of 3e38)
        b.rope_shift(); b.select(); torch.cuda.synchronize()
        got.append(b.scores.cpu().double())
    entries = plan_list_of(b.ws_select, up(w.n_tok * hq * 4) + up(w.n_tok * 4), w.n_tok, len(w.segments), w.n_requests)
    assert sorted(entries) == [(r, k) for r in range(w.n_requests) for k in range(tiles[r])]
    # (the bounds of assert_scores_agree and, for the sums of many keys, of test_scores_in_two_key_streams)
    sums, d = 4 * math.sqrt(max(sum(lens[i] for i in c) for c in chunks)) * 2.0 ** -24, (got[1] - got[0]).abs()
    assert float(d.max()) <= 2.0 ** -8 * 16 / math.sqrt(128) / 16 / hq + sums and float(d.pow(2).mean().sqrt()) <= 1e-6 + sums


@pytest.mark.parametrize("n", [8192, 8193])
@pytest.mark.parametrize("frac", [0.1, 0.6])
def test_selection_behind_wide_scores_of_eight_heads_per_kv_head(n, frac):
    # (eight wavefronts: keys stay in registers up to 8192 tokens.)  Every other token finds nothing in the chunk before: ties
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("topn8", "bf16", 8, 1, 128, 5.0e5, [40, n], [0, 0], [W.RequestSpec([0, 1], [0.2, frac], 3)], 1.0 / math.sqrt(128), seed=157)
    w.q[::2, :, 60:64] = 2.0
    w.q[:, :, 124:128] = 0.0
    for blk in w.store_tab[w.store_tab_off[0]: w.store_tab_off[1]]:
        w.k_store[blk, :, :, 60:64] = -141.0
        w.k_store[blk, :, :, 124:128] = 0.0
    b = DeviceBatch(w, impl=P.CC_IMPL_MFMA_WIDE, poison=True)
    b.rope_shift(); b.select(); torch.cuda.synchronize()
    scores = b.scores.cpu().numpy().astype(np.float64)
    sg = H.chunk_segments(w, 0)[1]
    own = scores[int(sg[W.SEG_TOK]): int(sg[W.SEG_TOK]) + n]
    assert (own == 0).sum() > n // 4 and (own > 0).sum() > n // 4
    assert np.array_equal(H.gpu_selection(w, b.sel_idx.cpu().numpy())[0][1], O.top_n(own, int(sg[W.SEG_NSEL])))


@pytest.mark.parametrize("op,n_out,n_in,rows", [
    ("linear", 64, 8192, 1), ("linear", 128, 5056, 17), ("linear", 256, 14336, 63), ("linear", 1024, 14336, 65),      # 64 x 64 and 64 x 128 tiles
    ("linear", 4096, 14336, 129), ("linear", 2048, 28672, 257), ("linear", 4096, 8256, 513),     # 128 x 128 up to 256 x 256
    ("linear", 8192, 14336, 2278),                               # whole rounds of the largest tile, the rest in parts
    ("qkv", 6144, 8192, 16), ("qkv", 6144, 14336, 300)])
def test_matrix_products_with_the_contraction_in_parts(op, n_out, n_in, rows):
    # stages that do and do not divide over the parts, row blocks one row short and one over, tiles whose rows end early
    import paper_2502_15734_amd as P
    g = torch.Generator(device="cuda").manual_seed(rows)
    rnd = lambda *s, sc=1.0: (torch.randn(*s, device="cuda", generator=g) * sc).to(torch.bfloat16)
    ctx = P.Context(32, 8, 128, 5.0e5, P.CC_BF16)
    x, w, res = rnd(rows, n_in), rnd(n_out, n_in, sc=n_in ** -0.5), rnd(rows, n_out)
    nbytes = ctx.qkv_project_workspace_bytes(rows, n_in) if op == "qkv" else ctx.linear_workspace_bytes(rows, n_in, n_out)
    assert 0 < nbytes <= 256 << 20
    room = torch.full((nbytes + 64,), 0xff, dtype=torch.uint8, device="cuda")        # (NaN in every place a part could leave out)
    def product(workspace):
        if op == "qkv":
            got = [torch.full((rows, n), float("nan"), dtype=torch.bfloat16, device="cuda") for n in (4096, 1024, 1024)]
            ctx.qkv_project(x, w, *got, workspace=workspace)
            return torch.cat(got, dim=1).float()
        y = res.clone()
        ctx.linear(x, w, y, residual=y, workspace=workspace)                     # (the residual may be the output)
        return y.float()
    want = x.double() @ w.double().t() + (0 if op == "qkv" else res.double())
    whole = product(torch.empty(0, dtype=torch.uint8, device="cuda"))            # no room: not split
    # half a unit in the last place of bf16, and fp32 sums of n_in products of size n_in^-1/2
    off = lambda got: float(((got - want).abs() - 2.0 ** -8 * want.abs()).max())
    # the room asked for, half of it (fewer parts or none), what the call takes by itself
    for workspace in (room[:nbytes], room[:nbytes // 32 * 16], None):
        got = product(workspace)
        assert off(got) <= 8 * n_in * 2.0 ** -24 * 4
        # no further from 64 bits than the whole contraction (both are roundings of nearly the same sums)
        assert float((got - want).norm()) <= 1.01 * float((whole - want).norm())
    torch.cuda.synchronize()
    assert bool((room[nbytes:] == 0xff).all())
    with pytest.raises(P.CacheCraftError):
        ctx.linear(x, w, res, workspace=room[8:])                                # not 16-byte aligned


@pytest.mark.parametrize("hq,hkv,lens,question,n_requests,parts", [
    (8, 2, [5], 40, 1, 1), (8, 2, [64, 0, 1, 130], 3, 2, 2), (8, 2, [2] * 254, 1, 1, 1), (8, 2, [1] * 255, 2, 1, 1), (8, 2, [3] * 300, 5, 1, 1),
    (8, 2, [700], 90, 3, 24), (8, 2, [210, 0, 1, 300, 5], 33, 2, 5), (8, 2, [1000, 0, 1, 3], 2, 1, 12), (64, 8, [2000] + [0, 1] * 130, 3, 1, 4),
    (32, 8, [300, 0, 30], 1, 1, 20), (64, 8, [1100], 2, 1, 32)])
def test_pair_masses_of_few_and_of_many_segments(hq, hkv, lens, question, n_requests, parts):
    # the masses are summed a segment's rows in parts (one part for every 128 pairs of a row and a head that a segment has on the average, up to 32), threads
    # side by side along the key segments: a segment with one key segment, segments without tokens, 255 to 301 of them (a workgroup has 256 threads); in one part,
    # and in several with fewer rows than parts, none at all, more
    from paper_2502_15734_amd.pipeline import DeviceBatch
    k = len(lens)
    assert parts == min(max((sum(lens) + question) * hq // (128 * (k + 1)), 1), 32)
    w = W.custom("pairs", "bf16", hq, hkv, 128, 5.0e5, lens * n_requests, [0] * (k * n_requests),
                 [W.RequestSpec(list(range(k * r, k * r + k)), [1.0] * k, question) for r in range(n_requests)], 1.0, seed=59)
    b = DeviceBatch(w, poison=True)
    b.rope_shift(); b.select(); b.gather()
    b.sparse_prefill_pairs()
    b.ws_prefill_pairs.fill_(0xff)                           # (NaN in every part that might be left out)
    pair, own, off = b.sparse_prefill_pairs()
    pair, own = pair.double().cpu(), own.double().cpu()
    pair2, own2, _ = b.chunk_attention()                     # by passes of its own over the segments
    torch.cuda.synchronize()
    # the weights of a row sum to 1: 8 heads' terms of up to (k + 1) segments in fp32
    for r in range(n_requests):
        for t in range(k + 1):
            rows = question if t == k else lens[t]
            at = int(off[r]) + t * (t + 1) // 2
            assert abs(float(pair[at:at + t + 1].sum()) - rows) <= 2.0 ** -20 * max(rows, 1) * (t + 2)
    # (both from products of the same bf16 queries and keys; the log-sum-exps, of up to 10, are fp32 and enter as exp: 2^-20 of a row each)
    rows_of = torch.tensor([float(question if t == k else lens[t]) for _ in range(n_requests) for t in range(k + 1) for _ in range(t + 1)])
    assert bool(((pair - pair2.double().cpu()).abs() <= 2.0 ** -9 * pair2.double().cpu() + 2.0 ** -17 * (rows_of + 1)).all())
    assert torch.equal(own, own2.double().cpu()) or float((own - own2.double().cpu()).abs().max()) <= 2.0 ** -9 * (question + max(lens, default=0))


@pytest.mark.parametrize("impl", ["AUTO", "MFMA_WIDE"])
@pytest.mark.parametrize("which,question", [(0, 32), (2, 32), (2, 31), (2, 1)])
def test_one_request_of_a_batch_leaves_the_safe_range(impl, which, question):
    # the second passes leave at once unless some row or token was flagged: only the first or only the last request's are, and the
    # list's last row is the last of a flag's 32, the first, in between
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    w = W.custom("one", "bf16", 8, 2, 128, 5.0e5, [64, 96] * 3, [0] * 6, [W.RequestSpec([2 * r, 2 * r + 1], [1.0, 1.0], question) for r in range(3)],
                 1.0 / math.sqrt(128), seed=29)
    w.q[:, :, 60:64] = 2.0
    w.q[:, :, 124:128] = 0.0
    blocks = w.store_tab[w.store_tab_off[2 * which]: w.store_tab_off[2 * which + 1]]
    first = which * (64 + 96 + question)
    for t in range(64):                                      # (logits around -100, as above)
        for keys, at in ((w.k_store, (blocks[t // 16], slice(None), t % 16)), (w.k_new, (first + t, slice(None)))):
            keys[at + (slice(60, 64),)] = -141.0
            keys[at + (slice(124, 128),)] = 0.0
    got = []
    for form in ("MFMA_NARROW", impl):
        b = DeviceBatch(w, impl=getattr(P, "CC_IMPL_" + form), poison=True)
        b.step(); torch.cuda.synchronize()
        n = w.n_q_tot
        got.append((b.out[:n].double(), b.lse[:n].double(), b.scores.double(), b.q_pos[:n].cpu()))
    assert torch.equal(got[0][3], got[1][3])                 # (everything is recomputed: the same rows)
    assert bool(torch.isfinite(got[1][0]).all()) and bool(torch.isfinite(got[1][1]).all())
    assert float((got[1][0] - got[0][0]).norm() / got[0][0].norm()) <= H.TOL["bf16"]
    rows = torch.arange(w.n_q_tot) // (64 + 96 + question)
    alone = (rows == which) & (got[0][3] < 64)               # rows that see such keys only: half a unit in the last place of four of them
    assert bool(((got[1][1] - got[0][1]).abs().cpu() <= torch.where(alone[:, None], 0.8, 2e-3)).all())
    assert float((got[1][2] - got[0][2]).abs().max()) <= 5e-5


@pytest.mark.parametrize("n", [1, 32, 33, 64, 97, 129, 192, 257, 320, 385, 449, 512, 609, 641, 705, 833])
def test_two_key_streams_of_few_blocks(n):
    # the streams' rings hold five 32-key blocks of K and four of V: less than that, as much, more, an odd tile, a last tile of one block or a part
    # of one; the by-product has its segments' ends in either stream
    import paper_2502_15734_amd as P
    from paper_2502_15734_amd.pipeline import DeviceBatch
    lens = [n // 3, n - n // 3]
    w = W.custom("rings", "bf16", 4, 1, 128, 5.0e5, lens, [0, 0], [W.RequestSpec([0, 1], [0.1, 0.05], 2)], 1.0, seed=n)
    b = DeviceBatch(w, poison=True)
    b.rope_shift(); b.select(); b.gather(); b.sparse_prefill(); torch.cuda.synchronize()
    sel = tuple(t.cpu().numpy()[: w.n_q_tot] for t in (b.sel_idx, b.q_row, b.q_pos, b.slot_map))
    s = DeviceBatch(w, impl=P.CC_IMPL_SCALAR, poison=True)
    s.rope_shift(); s.set_selection(*sel); s.gather(); s.sparse_prefill(); torch.cuda.synchronize()
    k = w.n_q_tot
    out, ref = b.out[:k].double(), s.out[:k].double()
    assert float((out - ref).norm() / ref.norm()) <= H.TOL["bf16"]
    # (bounds as above: six roundings of the query in a row that sees a single key)
    assert float((b.lse[:k] - s.lse[:k]).abs().max()) <= 6 * 2.0 ** -9 / 3.0 ** 0.5
    out1, lse1 = b.out[:k].clone(), b.lse[:k].clone()
    mass, want = b.sparse_prefill_mass(), s.sparse_prefill_mass()
    torch.cuda.synchronize()
    assert torch.equal(out1, b.out[:k]) and torch.equal(lse1, b.lse[:k])
    assert float((mass - want).abs().max()) <= 2.0 ** -7          # (two question rows; their logits within 6.8e-3, see above)
