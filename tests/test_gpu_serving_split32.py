"""GPU parity of the last query block's forward at block size 32 (bf16) where four wavefronts share its walk: fewer tiles than wavefronts,
lists past 64 entries, windows of more than 64 tiles, padding in any share, logits that send the block through the walk again."""
import math

import numpy as np
import pytest
import torch

import oracle
from gpu_util import TOL, Dev, assert_close, host, params
from paper_2512_13368_amd import binding as B
from paper_2512_13368_amd.inputs import WORKLOADS, make_inputs, with_shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,topk,window,sblk,amp,edit", [
    (32 * 17, 4, 64, 0, 1, None),           # the shortest history and the shortest list that are shared
    (32 * 40 + 5, 16, 128, 0, 1, None),     # a ragged last block
    (32 * 33, 9, 700, 0, 1, None),          # more window tiles than list entries
    (32 * 90, 70, 2200, 0, 1, None),        # more than 64 of either
    (32 * 21 + 30, 12, 100, 32, 1, None),   # all of Eq. 15
    (32 * 21 + 30, 12, 100, 1, 1, None),
    (32 * 20, 10, 20, 0, 1, "none"),        # two short-term tiles alone: wavefronts without any
    (32 * 20, 10, 64, 0, 1, "holes"),
    (32 * 22 + 28, 9, 100, 0, 512, None),   # logits in the hundreds (a scale that log2(e) turns into a power of two: Q stays exact)
])
def test_last_block_in_four_wavefronts(L, topk, window, sblk, amp, edit):
    w = with_shape(WORKLOADS["cfg3"], name=f"split32-L{L}-k{topk}-w{window}-s{sblk}-{edit}-x{amp}", B=5, H=3, L=L, topk=topk, window=window,
                   len_lo=1, len_hi=L, stis_block=sblk, seed=7100 + L + topk)
    x = make_inputs(w)
    x.valid_len[:4] = [L, max(1, L - 70), min(L, 20), 0]
    scale = {} if amp == 1 else {"scale": amp * math.log(2.0)}
    extra = {} if amp == 1 else {"softmax_scale": amp * math.log(2.0)}
    dv, p = Dev(x), params(w, last_block_only=1, save_for_bwd=1, **extra)
    sel = B.select_blocks(params(w), dv.Q, dv.K, dv.vl)
    last = sel[:, :, -1]
    if edit == "none":
        last[:] = -1
    elif edit == "holes":
        last[:, :, ::2] = -1
        last[:, :, 1] = w.NB + 3
    fill = lambda *s: torch.full(s, 3.0, device="cuda")
    f = B.FwdOut(torch.full_like(dv.Q, 3.0), fill(w.B, w.H, L, w.d), fill(w.B, w.H, L, w.d), fill(w.B, w.H, L), fill(w.B, w.H, L))
    B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, out=f)
    torch.cuda.synchronize()
    lo = (w.NB - 1) * 32
    fr = oracle.attn_fwd(x.Q, x.K, x.V, x.valid_len, sel.cpu().numpy(), x.gate_w, x.gate_b, 32, topk, window, stis_block=sblk, **scale)
    for name in ("O", "o_lt", "o_st", "lse_lt", "lse_st"):
        got = getattr(f, name)
        assert bool((got[:, :, :lo] == 3.0).all()), name
        ref = getattr(fr, name).reshape(got.shape)[:, :, lo:]
        assert_close(host(got[:, :, lo:]), np.ascontiguousarray(ref), TOL["bf16"], name)
