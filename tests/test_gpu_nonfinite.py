"""Values that are not finite in the small-head kernels (d in {8, 16, 32}, block 8 or 16): they reach every output that
depends on them, and no other."""
import pytest
import torch

from gpu_util import Dev, params
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
