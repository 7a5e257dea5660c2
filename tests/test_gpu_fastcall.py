"""The native marshalling of the hot calls against the Python path: with every buffer given by the caller a call goes
through the former, with any left out through the latter; results, error codes and messages are the same."""
import pytest
import torch

from gpu_util import Dev, params
from paper_2512_13368_amd import binding as B
from paper_2512_13368_amd.inputs import WORKLOADS, make_inputs, rope_tables, with_shape

pytestmark = pytest.mark.gpu


def _fwd_like(f):
    return B.FwdOut(*(torch.full_like(t, 7.0) for t in (f.O, f.o_lt, f.o_st, f.lse_lt, f.lse_st)))


def _bwd_like(g):
    return B.BwdOut(*(torch.full_like(t, 7.0) for t in (g.dQ, g.dK, g.dV, g.d_gate_w, g.d_gate_b)))


def _equal(a, b, names):
    for n in names:
        assert torch.equal(getattr(a, n), getattr(b, n)), n


def _ws(count):
    return torch.empty(max(16, count), dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("name,shape", [("cfg2", dict(B=5, H=2, L=70, len_lo=3, len_hi=70)),
                                        ("cfg3", dict(B=3, H=2, L=200, len_lo=20, len_hi=200))])
def test_both_paths_agree(name, shape):
    w = with_shape(WORKLOADS[name], name=f"fast-{name}", **shape)
    dv, p = Dev(make_inputs(w, want_dO=True)), params(w, save_for_bwd=1)
    cos, sin = (torch.from_numpy(t).cuda() for t in rope_tables(w.L, w.d))
    ws_s, ws_b = _ws(B.workspace_bytes(p, B.WS_SELECT)), _ws(B.workspace_bytes(p, B.WS_BWD))
    side = torch.cuda.Stream()
    outs = ("O", "o_lt", "o_st", "lse_lt", "lse_st")
    grads = ("dQ", "dK", "dV", "d_gate_w", "d_gate_b")

    sel = B.select_blocks(p, dv.Q, dv.K, dv.vl)
    assert torch.equal(B.select_blocks(p, dv.Q, dv.K, dv.vl, sel=torch.full_like(sel, 9), ws=ws_s), sel)
    rot = B.rope_select_blocks(p, dv.Q, dv.K, cos, sin, dv.vl)
    for a, b in zip(B.rope_select_blocks(p, dv.Q, dv.K, cos, sin, dv.vl, *(torch.zeros_like(t) for t in rot), ws=ws_s), rot):
        assert torch.equal(a, b)
    f = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb)
    with torch.cuda.stream(side):
        side.wait_stream(torch.cuda.default_stream())
        f2 = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, out=_fwd_like(f))
    side.synchronize()
    _equal(f, f2, outs)
    for rope in (None, (cos, sin)):
        g = B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO, rope=rope)
        g2 = B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO, out=_bwd_like(g), ws=ws_b,
                        stream=torch.cuda.current_stream(), rope=rope)
        torch.cuda.synchronize()
        _equal(g, g2, grads)

    with pytest.raises(ValueError, match="^K: expected contiguous"):
        B.attn_fwd(p, dv.Q, dv.K[:, :1], dv.V, dv.vl, sel, dv.gw, dv.gb, out=f2)
    with pytest.raises(ValueError, match="^sel: expected contiguous"):
        B.select_blocks(p, dv.Q, dv.K, dv.vl, sel=sel.long(), ws=ws_s)
    for call in (lambda: B.select_blocks(p, dv.Q, dv.K, dv.vl, sel=sel, ws=ws_s[:16]),
                 lambda: B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO, out=g2, ws=ws_b[:16])):
        with pytest.raises(B.BlossomError, match=B.strerror(-6)[:20]):
            call()
    torch.cuda.synchronize()


def test_both_paths_agree_per_position_and_projection():
    n, H, G, L, d = 3, 4, 2, 60, 16
    g = torch.Generator(device="cuda").manual_seed(3)
    new = lambda *s: torch.randn(s, generator=g, device="cuda")
    p = B.Params(n, H, L, d, 16, 3, 8, B.F32, stis_mode=1, stis_block=1)
    Q, dO, K, V = new(n, H, L, d), new(n, H, L, d), new(n, G, L, d), new(n, G, L, d)
    vl = torch.tensor([60, 31, 0], dtype=torch.int32, device="cuda")
    gw, gb = new(H, 2 * d), new(H)
    sel = B.select_positions(p, G, 32, 16, Q, K, vl)
    ws = _ws(B.select_positions_workspace_bytes(p, G, 32, 16))
    assert torch.equal(B.select_positions(p, G, 32, 16, Q, K, vl, sel_pos=torch.zeros_like(sel), ws=ws), sel)
    f = B.attn_fwd_positions(p, G, Q, K, V, vl, sel, gw, gb, want_branches=True)
    f2 = B.attn_fwd_positions(p, G, Q, K, V, vl, sel, gw, gb, out=_fwd_like(f))
    _equal(f, f2, ("O", "o_lt", "o_st", "lse_lt", "lse_st"))
    b = B.attn_bwd_positions(p, G, Q, K, V, vl, sel, gw, gb, f, dO)
    b2 = B.attn_bwd_positions(p, G, Q, K, V, vl, sel, gw, gb, f, dO, out=_bwd_like(b), ws=_ws(B.workspace_bytes(p, B.WS_BWD)))
    _equal(b, b2, ("dQ", "dK", "dV", "d_gate_w", "d_gate_b"))
    W, prev, gamma, beta = new(64, H * d), new(n, L, 64), new(64), new(64)
    S, mean, rstd = B.out_proj_ln(p, 64, f.O, W, prev, gamma, beta, 1e-5, want_stats=True)
    S2, mean2, rstd2 = B.out_proj_ln(p, 64, f.O, W, prev, gamma, beta, 1e-5, S=torch.zeros_like(S), want_stats=True)
    torch.cuda.synchronize()
    assert torch.equal(S, S2) and torch.equal(mean, mean2) and torch.equal(rstd, rstd2)
