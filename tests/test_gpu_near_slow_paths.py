"""The repeats of the small heads' near form, where its walks cover several words of tiles, stream their tiles, or serve several query heads:
logits that one exponential cannot take, keys and values that are not finite in any word's tiles, padding that holds anything.  With
them the streamed shapes in bf16 storage, ordinary values too."""
import numpy as np
import pytest
import torch

import oracle
import test_gpu_nonfinite as nonfinite
from gpu_util import TOL, Dev, assert_close, host, params, to_dev
from paper_2512_13368_amd import binding as B
from paper_2512_13368_amd.inputs import WORKLOADS, make_inputs, round_to_bf16, with_shape
from test_gpu_parity import run_case

pytestmark = pytest.mark.gpu

# dtype, d, block, length, mask block
STREAMED = [("fp32", 8, 16, 1100, 1), ("fp32", 16, 16, 1100, 0), ("fp32", 8, 8, 1043, 1), ("fp32", 32, 16, 1100, 1), ("bf16", 8, 16, 1100, 1),
            ("bf16", 16, 16, 1060, 1), ("bf16", 32, 16, 1100, 1), ("bf16", 32, 8, 1050, 0)]


@pytest.mark.parametrize("dtype,d,b,L,sblk", STREAMED)
@pytest.mark.parametrize("amp", [1, 32])   # 32: base-2 logits beyond 60 in every tile
def test_streamed_over_several_words(dtype, d, b, L, sblk, amp):
    w = with_shape(WORKLOADS["cfg2"], name=f"near-words-{dtype}-d{d}-b{b}-L{L}-s{sblk}-x{amp}", B=3, H=2, L=L, d=d, block=b, topk=6, window=9,
                   dtype=dtype, len_lo=1, len_hi=L, stis_block=sblk, backward=False, seed=6300 + d + L)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:] = [L, L - 21, L - 16 * 9 - 3]
    x.Q *= np.float32(amp)
    run_case(w, x=x, backward=True, gate_scale=0.4)


@pytest.mark.parametrize("shape", STREAMED)
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_padding_may_hold_anything(shape, value):
    dtype, d, b, L, sblk = shape
    nonfinite.test_padding_may_hold_anything((dtype, d, b, 3, 2, L, sblk, False), value)


def _masks_of(w, sel, r, h, n, sblk, per_position=False):
    M_lt, M_st = oracle.build_masks(w["L"], w["b"], w["k"], w["window"], n, sel[r, h], sblk, False, per_position)
    return (M_lt | M_st).astype(bool)


@pytest.mark.parametrize("dtype,d,b,L,sblk", STREAMED)
@pytest.mark.parametrize("where", ["K", "V"])
@pytest.mark.parametrize("at", [70, -10])   # in the first word's tiles, listed by blocks of the others; beside the last rows
def test_a_row_of_nan_in_another_word(dtype, d, b, L, sblk, where, at):
    w = with_shape(WORKLOADS["cfg2"], name=f"near-nan-{dtype}-d{d}-b{b}-L{L}-{where}{at}", B=2, H=2, L=L, d=d, block=b, topk=4, window=9,
                   dtype=dtype, len_lo=L, len_hi=L, stis_block=sblk, seed=6500 + d + L)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:] = [L, L - 37]
    print(w.name, flush=True)
    dv, p = Dev(x), params(w, save_for_bwd=1)
    sel = B.select_blocks(p, dv.Q, dv.K, dv.vl)
    at = at % L
    blocks = torch.arange(w.NB, device="cuda")
    sel[:, :, :, -1] = torch.where((blocks > at // b + 2) & (blocks % 3 > 0), at // b, sel[:, :, :, -1])   # two blocks of three list it last
    clean = nonfinite._run(dv, p, sel)
    r, h = 1, 1
    getattr(dv, where)[r, h, at] = float("nan")
    got = nonfinite._run(dv, p, sel)
    seen = _masks_of(dict(L=L, b=b, k=4, window=9), sel.cpu().numpy(), r, h, x.valid_len[r], sblk)
    queries = seen[:, at]
    keys = seen[queries].any(0) | (np.arange(L) == at)
    assert queries.sum() > 8
    for name, lost in (("O", queries), ("dQ", queries), ("dV", keys), ("dK", keys)):
        assert bool(got[name][r, h][torch.from_numpy(lost).cuda()].isnan().all()), name
        assert_close(host(got[name][r, h])[~lost], host(clean[name][r, h])[~lost], TOL[dtype], name)
        got[name][r, h], clean[name][r, h] = 0.0, 0.0
        assert torch.equal(got[name], clean[name]), name


# dtype, query heads, key/value heads, length, d, mask block
POSITIONS = [("fp32", 8, 4, 200, 8, 1), ("fp32", 8, 2, 640, 8, 1), ("fp32", 4, 2, 500, 16, 1), ("bf16", 4, 2, 360, 32, 0), ("bf16", 8, 2, 90, 16, 1)]


def _positions(dtype, H, G, L, d, sblk, amp=1.0):
    rng = np.random.default_rng(6700 + L + d)
    n = 3
    Q, K, V, dO = (rng.standard_normal((n, heads, L, d)).astype(np.float32) for heads in (H, G, G, H))
    Q *= np.float32(amp)
    if dtype == "bf16":
        Q, K, V, dO = (round_to_bf16(t) for t in (Q, K, V, dO))
    gw, gb = (rng.standard_normal((H, 2 * d)) * 0.3).astype(np.float32), (rng.standard_normal(H) * 0.5).astype(np.float32)
    vl = np.array([L, L - 21, min(L, 40)], np.int32)
    print(f"near positions {dtype} H{H} G{G} L{L} d{d} s{sblk} x{amp}", flush=True)
    p = B.Params(n, H, L, d, 16, 4, 8, B.F32 if dtype == "fp32" else B.BF16, stis_mode=int(sblk > 0), stis_block=sblk)
    dev = [to_dev(t, dtype) for t in (Q, K, V, dO)]
    small = [torch.from_numpy(t).cuda() for t in (vl, gw, gb)]
    sel = B.select_positions(p, G, 32, 16, dev[0], dev[1], small[0])

    def run():
        f = B.attn_fwd_positions(p, G, *dev[:3], small[0], sel, *small[1:], want_branches=True)
        g = B.attn_bwd_positions(p, G, *dev[:3], small[0], sel, *small[1:], f, dev[3])
        torch.cuda.synchronize()
        return {"O": f.O, "o_lt": f.o_lt, "o_st": f.o_st, "dQ": g.dQ, "dK": g.dK, "dV": g.dV, "d_gate_w": g.d_gate_w, "d_gate_b": g.d_gate_b}

    return (Q, K, V, dO, vl, gw, gb), dev, sel, run


@pytest.mark.parametrize("case", POSITIONS)
def test_large_logits_per_position(case):
    dtype, H, G, L, d, sblk = case
    (Q, K, V, dO, vl, gw, gb), _, sel, run = _positions(*case, amp=32.0)
    got = run()
    rep = lambda t: np.repeat(t, H // G, axis=1)
    args = (Q, rep(K), rep(V), vl, np.ascontiguousarray(rep(sel.cpu().numpy())), gw, gb)
    fr = oracle.attn_fwd(*args, 16, 4, 8, stis_block=sblk, per_position=True)
    gr = oracle.attn_bwd(*args, dO, 16, 4, 8, stis_block=sblk, per_position=True)
    over = lambda t: t.reshape(3, G, H // G, L, d).sum(2)
    for name, ref in (("O", fr.O), ("o_lt", fr.o_lt), ("o_st", fr.o_st), ("dQ", gr.dQ), ("dK", over(gr.dK)), ("dV", over(gr.dV))):
        assert_close(host(got[name]), ref.reshape(got[name].shape), TOL[dtype], name)


@pytest.mark.parametrize("case", POSITIONS)
def test_what_is_not_finite_per_position(case):
    dtype, H, G, L, d, sblk = case
    (_, _, _, _, vl, _, _), dev, sel, run = _positions(*case)
    clean = run()
    pad = (torch.arange(L, device="cuda")[None, :] < L - torch.from_numpy(vl).cuda()[:, None])[:, None, :, None]
    for t in dev:
        t.masked_fill_(pad, float("nan"))
    for name, t in run().items():
        assert_close(host(t), host(clean[name]), TOL[dtype], name)
    # a value row of NaN: the rows of its group's query heads that see it, and no others
    r, kv, at = 1, 1, L - 35
    dev[2][r, kv, at] = float("nan")
    got, rows = run(), sel.cpu().numpy()
    for h in range(H):
        seen = _masks_of(dict(L=L, b=16, k=4, window=8), rows, r, h // (H // G), vl[r], sblk, True)[:, at] & (h // (H // G) == kv)
        for name in ("O", "dQ"):
            assert bool(got[name][r, h][torch.from_numpy(seen).cuda()].isnan().all()), (name, h)
            assert_close(host(got[name][r, h])[~seen], host(clean[name][r, h])[~seen], TOL[dtype], (name, h))
    for name in ("dK", "dV"):
        assert bool(got[name][r, kv, at].isnan().all()), name
        assert_close(host(got[name][[0, 2]]), host(clean[name][[0, 2]]), TOL[dtype], name)
