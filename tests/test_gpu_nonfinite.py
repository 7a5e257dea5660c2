"""Values that are not finite in the small-head kernels (d in {8, 16, 32}, block 8 or 16) and in the scalar ones: they reach
every output that depends on them, and no other."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import TOL, Dev, assert_close, host, params
from paper_2512_13368_amd import binding as B
from paper_2512_13368_amd.inputs import WORKLOADS, make_inputs, with_shape

pytestmark = pytest.mark.gpu


def _valid(w, x):
    """[B, L] bool: the valid positions."""
    return torch.arange(w.L, device="cuda")[None, :] >= w.L - torch.from_numpy(x.valid_len).cuda()[:, None]


@pytest.mark.parametrize("where", ["gate_b", "gate_w"])
@pytest.mark.parametrize("d,b,L", [(32, 16, 90), (16, 8, 513), (8, 16, 800)])  # a head in LDS; streamed; streamed at d = 8
def test_nan_gate_is_not_swallowed(where, d, b, L):
    w = with_shape(WORKLOADS["cfg2"], name=f"nan-{where}-d{d}", B=2, H=3, L=L, d=d, block=b, topk=3, window=b, len_lo=5, len_hi=L,
                   seed=3100 + d)
    x = make_inputs(w, want_dO=True)
    x.valid_len[0] = L
    dv, p = Dev(x), params(w, save_for_bwd=1)
    (dv.gb if where == "gate_b" else dv.gw[:, 3])[1] = float("nan")
    sel = B.select_blocks(p, dv.Q, dv.K, dv.vl)
    f = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb)
    g = B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO)
    torch.cuda.synchronize()
    valid = _valid(w, x)
    for name, t in (("O", f.O), ("dQ", g.dQ), ("dV", g.dV)):
        assert bool(t[:, 1][valid].isnan().all()), name
        assert bool(t[:, ::2].isfinite().all()), name
    assert bool(f.o_lt.isfinite().all()) and bool(f.o_st.isfinite().all())  # (the branches come before the gate)
    assert bool(g.d_gate_w[1].isnan().all()) and bool(g.d_gate_b[1].isnan())
    assert bool(g.d_gate_w[::2].isfinite().all()) and bool(g.d_gate_b[::2].isfinite().all())


# a head in LDS (one, or beyond 2048 heads overlaid buffers); streamed; scalar; both storage types, all three short-term masks
SHAPES = [("fp32", 32, 16, 3, 2, 90, 0, False), ("bf16", 16, 8, 257, 8, 60, 1, False), ("fp32", 8, 8, 3, 2, 1043, 5, True),
          ("bf16", 32, 16, 3, 2, 300, 2, True), ("fp32", 16, 16, 3, 2, 530, 1, False),
          ("fp32", 64, 16, 3, 2, 90, 1, False), ("bf16", 64, 32, 3, 2, 150, 4, True)]


def _case(dtype, d, b, rows, H, L, sblk, bidir):
    w = with_shape(WORKLOADS["cfg2"], name=f"nonfinite-{dtype}-d{d}-b{b}-L{L}", B=rows, H=H, L=L, d=d, block=b, topk=3,
                   window=b // 2 + 1, dtype=dtype, qkv_scaled=(dtype == "bf16"), len_lo=1, len_hi=L, stis_block=sblk, bidir=bidir,
                   seed=3300 + d + b + L)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:3] = [L - b // 2 - 1, L - 2 * b - 3, min(L, b // 2 + 1)]  # rows that begin inside a tile
    print(w.name, flush=True)
    return w, x, Dev(x), params(w, save_for_bwd=1)


def _run(dv, p, sel):
    f = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb)
    g = B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO)
    torch.cuda.synchronize()
    return {"O": f.O, "o_lt": f.o_lt, "o_st": f.o_st, "lse_lt": f.lse_lt, "lse_st": f.lse_st, "dQ": g.dQ, "dK": g.dK, "dV": g.dV,
            "d_gate_w": g.d_gate_w, "d_gate_b": g.d_gate_b}


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("value", [float("nan"), float("inf"), -1e38])
def test_padding_may_hold_anything(shape, value):
    w, x, dv, p = _case(*shape)
    clean_sel = B.select_blocks(p, dv.Q, dv.K, dv.vl)
    clean = _run(dv, p, clean_sel)
    pad = ~_valid(w, x)[:, None, :, None]
    for t in (dv.Q, dv.K, dv.V, dv.dO):
        t.masked_fill_(pad, value)
    sel = B.select_blocks(p, dv.Q, dv.K, dv.vl)
    assert torch.equal(sel, clean_sel)
    for name, t in _run(dv, p, sel).items():
        assert_close(host(t), host(clean[name]), TOL[w.dtype], name)
    if not w.bidir:
        dense, _ = B.dense_causal_fwd(p, dv.Q, dv.K, dv.V, dv.vl)
        assert bool(dense.isfinite().all())


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("where", ["Q", "K", "V", "dO"])
def test_a_row_of_nan_reaches_what_depends_on_it(shape, where):
    w, x, dv, p = _case(*shape)
    sel = B.select_blocks(p, dv.Q, dv.K, dv.vl)
    clean = _run(dv, p, sel)
    r, h, at = 1, 1, w.L - w.block - 2  # a valid row with valid rows before and behind it in its tile
    getattr(dv, where)[r, h, at] = float("nan")
    got = _run(dv, p, sel)
    M_lt, M_st = oracle.build_masks(w.L, w.block, w.topk, w.window, x.valid_len[r], sel[r, h].cpu().numpy(), w.stis_block, w.bidir)
    seen = (M_lt | M_st).astype(bool)  # [query, key]
    queries = seen[:, at] if where in "KV" else np.arange(w.L) == at  # the rows whose own quantities are lost
    keys = seen[queries].any(0) | (np.arange(w.L) == at if where in "KV" else False)
    lost = {"O": queries if where != "dO" else None, "dQ": queries, "dV": keys, "dK": keys}
    for name in ("O", "dQ", "dK", "dV"):
        bad, ok = lost[name], np.ones(w.L, bool) if lost[name] is None else ~lost[name]
        assert bad is None or bool(got[name][r, h][torch.from_numpy(bad).cuda()].isnan().all()), name
        assert_close(host(got[name][r, h])[ok], host(clean[name][r, h])[ok], TOL[w.dtype], name)
    got["d_gate_w"][h] = got["d_gate_b"][h] = 0.0  # (sums over the rows)
    clean["d_gate_w"][h] = clean["d_gate_b"][h] = 0.0
    for name in clean:  # every other head: the same bits
        if name[:2] != "d_":
            got[name][r, h], clean[name][r, h] = 0.0, 0.0
        assert torch.equal(got[name], clean[name]), name


def test_padding_may_hold_anything_with_shared_key_heads():
    n, H, G, L, d = 3, 8, 2, 100, 16
    gen = torch.Generator(device="cuda").manual_seed(5)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda")
    p = B.Params(n, H, L, d, 16, 3, 8, B.F32, stis_mode=1, stis_block=1)
    Q, dO, K, V, gw, gb = new(n, H, L, d), new(n, H, L, d), new(n, G, L, d), new(n, G, L, d), new(H, 2 * d), new(H)
    vl = torch.tensor([91, 57, 5], dtype=torch.int32, device="cuda")
    sel = B.select_positions(p, G, 32, 16, Q, K, vl)

    def run():
        f = B.attn_fwd_positions(p, G, Q, K, V, vl, sel, gw, gb, want_branches=True)
        g = B.attn_bwd_positions(p, G, Q, K, V, vl, sel, gw, gb, f, dO)
        torch.cuda.synchronize()
        return f.O, g.dQ, g.dK, g.dV, g.d_gate_w, g.d_gate_b

    clean = run()
    pad = (torch.arange(L, device="cuda")[None, :] < L - vl[:, None])[:, None, :, None]
    for t in (Q, dO, K, V):
        t.masked_fill_(pad, float("nan"))
    for got, want in zip(run(), clean):
        assert_close(host(got), host(want), TOL["fp32"])
