"""GPU parity of the small-head kernels' near form (causal, Eq. 15 left out or with mask block 1, windows of up to 17 positions): the
tile before the row's own, the first valid tile in every role a walk gives it, lists without the own block or with more than 64
entries, word boundaries of the tile lists, and the lengths of a row's history at which there is nothing to walk."""
import numpy as np
import pytest

from paper_2512_13368_amd.inputs import WORKLOADS, make_inputs, with_shape
from test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


def _edit(sel):
    """Every third query block loses its own entry, every other third has its list reversed and names a later block and one past the end."""
    NB = sel.shape[2]
    for I in range(NB):
        row = sel[:, :, I]
        if I % 3 == 1:
            row[(row == I) & ((row >= 0).sum(-1, keepdims=True) >= 2)] = -1
        elif I % 3 == 2:
            sel[:, :, I] = row[..., ::-1].copy()
            free = sel[:, :, I, 0] < 0
            sel[:, :, I, 0][free] = NB + 64
    return sel


@pytest.mark.parametrize("d,b,L,topk,window,sblk,dtype", [
    (16, 16, 15, 2, 1, 1, "fp32"),       # one tile, the window the position itself
    (8, 16, 17, 2, 17, 0, "fp32"),       # a second tile of one row, the longest window
    (32, 8, 100, 3, 17, 1, "fp32"),      # two blocks to a tile, the last tile half empty
    (16, 16, 208, 20, 8, 1, "bf16"),     # more entries than blocks
    (32, 16, 197, 4, 16, 1, "bf16"),
    (8, 16, 1025, 4, 8, 1, "fp32"),      # tile 64: the tile before the row's own is in another word
    (16, 16, 1040, 70, 2, 0, "fp32"),    # lists of more than 64 entries
    (32, 16, 1100, 3, 8, 1, "fp32"),
    (16, 8, 1056, 5, 9, 1, "fp32"),
    (8, 8, 2070, 6, 17, 1, "bf16"),      # 130 tiles: three words
])
def test_near_form(d, b, L, topk, window, sblk, dtype):
    w = with_shape(WORKLOADS["cfg2"], name=f"near-d{d}-b{b}-L{L}-k{topk}-w{window}-s{sblk}-{dtype}", B=8, H=2, L=L, d=d, block=b, topk=topk,
                   window=window, dtype=dtype, qkv_scaled=(dtype == "bf16"), len_lo=0, len_hi=L, stis_block=sblk, seed=5100 + L + topk)
    x = make_inputs(w, want_dO=True)
    # full; padding that ends inside the first, the second and the last tile; whole tiles of padding; one item; none
    x.valid_len[:7] = [L, max(L - 5, 1), max(L - 23, 1), min(L, 7), max(L - 64, 1), 1, 0]
    run_case(w, x=x, backward=True, gate_scale=0.4, sel_edit=_edit)


@pytest.mark.parametrize("L,B_", [(40, 3), (200, 700)])   # eight wavefronts to a head; four, and shared buffers
def test_large_logits_in_the_near_form(L, B_):
    w = with_shape(WORKLOADS["cfg2"], name=f"near-sharp-L{L}", B=B_, H=3, L=L, d=16, block=16, topk=3, window=8, len_lo=1, len_hi=L,
                   stis_block=1, backward=False, seed=5300 + L)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:2] = [L, max(1, L - 21)]
    x.Q *= np.float32(30)
    run_case(w, x=x, pairs=None if B_ < 64 else [0, 1, 3, 1001, B_ * 3 - 1], backward=True, gate_scale=0.4)
