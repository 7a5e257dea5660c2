"""GPU parity of the bf16 forward that walks the tiles of both branches once, at the edges of its tile lists: selections
without the own block, with entries in any order and past the 64 of a wavefront, windows of more than 64 tiles, logits
whose exponentials leave fp32's range without a reference, every short-term mask."""
import math

import pytest
import torch

from gpu_util import Dev, params
from paper_2512_13368_amd import binding as B
from paper_2512_13368_amd.inputs import WORKLOADS, make_inputs, with_shape
from test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


def _edit(sel):
    """Every third query block loses its own entry (where others remain), every other third has its list reversed."""
    for I in range(sel.shape[2]):
        row = sel[:, :, I]
        if I % 3 == 1:
            row[(row == I) & ((row >= 0).sum(-1, keepdims=True) >= 2)] = -1
        elif I % 3 == 2:
            sel[:, :, I] = row[..., ::-1].copy()
    return sel


@pytest.mark.parametrize("b", [32, 64])
@pytest.mark.parametrize("L,topk,window,sblk,amp,edit", [
    (17, 2, 9, 0, 1, False),          # one ragged block
    (300, 3, 1, 0, 1, True),          # a window of one key
    (500, 5, 64, 0, 1, True),
    (500, 4, 40, 64, 1, True),        # all of Eq. 15 with the mask block of the tile (64) or larger (32: scalar kernels)
    (500, 4, 40, 1, 1, True),         # ... and element by element
    (700, 4, 100, 0, 512, True),       # logits in the hundreds (a scale that log2(e) turns into a power of two: Q stays exact)
    (400, 3, 70, 1, 1024, False),
    (2300, 70, 2200, 0, 1, False),    # 72 blocks of 32: 70 list entries, 70 window tiles
])
def test_one_walk_for_both_branches(b, L, topk, window, sblk, amp, edit):
    w = with_shape(WORKLOADS["cfg3"], name=f"walk-b{b}-L{L}-k{topk}-w{window}-s{sblk}-x{amp}", B=3, H=2, L=L, block=b, topk=topk,
                   window=window, len_lo=1, len_hi=L, stis_block=sblk, backward=False, seed=2600 + L + topk)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:2] = [L, max(1, L - b - 3)]
    pairs = [0, 1, 2, 5] if L > 1000 else None
    run_case(w, x=x, pairs=pairs, backward=amp == 1, gate_scale=0.4, scale=None if amp == 1 else amp * math.log(2.0),
             sel_edit=_edit if edit else None)


def test_an_empty_list_does_not_send_a_block_through_the_walk_again():
    # no selected block at all: the long-term outputs are zeros, and the short-term ones are those of the one walk, bit for bit
    # (a second walk would take its exponentials against row maxima)
    w = with_shape(WORKLOADS["cfg3"], name="walk-empty-list", B=3, H=2, L=300, topk=3, len_lo=1, len_hi=300, seed=2650)
    x = make_inputs(w)
    x.valid_len[:2] = [300, 77]
    dv, p = Dev(x), params(w, save_for_bwd=1)
    sel = torch.full((w.B, w.H, w.NB, w.topk), -1, dtype=torch.int32, device="cuda")
    empty = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb)
    sel[..., 1] = torch.arange(w.NB, device="cuda")
    own = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb)
    torch.cuda.synchronize()
    assert not bool(empty.o_lt.any()) and not bool(empty.lse_lt.any()) and bool(own.o_lt.any())
    assert torch.equal(empty.o_st, own.o_st) and torch.equal(empty.lse_st, own.lse_st)
