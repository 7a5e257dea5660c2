"""GPU parity of the last query block's forward at block size 64 (bf16) where its tiles are shared out over three groups of wavefronts:
lists of every length down to an empty half, short-term walks longer than the list, padding in any of the groups' tiles."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import TOL, Dev, assert_close, host, params
from paper_2512_13368_amd import binding as B
from paper_2512_13368_amd.inputs import WORKLOADS, make_inputs, with_shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,topk,window,sblk,edit", [
    (64 * 8, 8, 64, 0, None),             # the shortest list that is shared
    (64 * 40 + 5, 16, 128, 0, None),      # a ragged last block
    (64 * 33, 9, 700, 0, None),           # more window tiles than either half of the list has
    (64 * 80, 70, 128, 0, None),          # more than 64 entries
    (64 * 21 + 60, 12, 100, 64, None),    # all of Eq. 15
    (64 * 21 + 60, 12, 100, 1, None),
    (64 * 12, 10, 64, 0, "one"),          # one entry: the third group has nothing
    (64 * 12, 10, 64, 0, "none"),         # no entry at all
    (64 * 12, 10, 64, 0, "holes"),
])
def test_last_block_in_three_groups(L, topk, window, sblk, edit):
    w = with_shape(WORKLOADS["cfg4"], name=f"split-L{L}-k{topk}-w{window}-s{sblk}-{edit}", B=5, H=3, L=L, topk=topk, window=window,
                   len_lo=1, len_hi=L, stis_block=sblk, seed=6100 + L + topk)
    x = make_inputs(w)
    x.valid_len[:4] = [L, max(1, L - 70), min(L, 30), 0]
    dv, p = Dev(x), params(w, last_block_only=1, save_for_bwd=1)
    sel = B.select_blocks(params(w), dv.Q, dv.K, dv.vl)
    last = sel[:, :, -1]
    if edit == "one":
        last[:, :, 1:] = -1
    elif edit == "none":
        last[:] = -1
    elif edit == "holes":
        last[:, :, ::2] = -1
        last[:, :, 1] = w.NB + 3
    fill = lambda *s: torch.full(s, 3.0, device="cuda")
    f = B.FwdOut(torch.full_like(dv.Q, 3.0), fill(w.B, w.H, L, w.d), fill(w.B, w.H, L, w.d), fill(w.B, w.H, L), fill(w.B, w.H, L))
    B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, out=f)
    torch.cuda.synchronize()
    lo = (w.NB - 1) * 64
    fr = oracle.attn_fwd(x.Q, x.K, x.V, x.valid_len, sel.cpu().numpy(), x.gate_w, x.gate_b, 64, topk, window, stis_block=sblk)
    for name in ("O", "o_lt", "o_st", "lse_lt", "lse_st"):
        got = getattr(f, name)
        assert bool((got[:, :, :lo] == 3.0).all()), name
        ref = getattr(fr, name).reshape(got.shape)[:, :, lo:]
        assert_close(host(got[:, :, lo:]), np.ascontiguousarray(ref), TOL["bf16"], name)
