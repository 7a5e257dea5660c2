"""GPU parity of the small heads' near form on both sides of the lines from which four wavefronts take a head instead of eight, and from
which heads are taken by length: every output of every head, the gate's sums among them."""
import pytest

import test_gpu_positions as positions
from paper_2512_13368_amd.inputs import WORKLOADS, make_inputs, with_shape
from test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,b,rows,H,lengths", [
    ("fp32", 8, 16, 129, 4, (62, 63, 103, 104)),     # 516 heads: by length from 63 on with four wavefronts, eight from 104 on
    ("fp32", 16, 8, 171, 4, (66, 67, 136, 137)),
    ("bf16", 16, 16, 257, 2, (61, 62, 102, 103)),
    ("fp32", 32, 16, 129, 4, (44, 45, 64, 65)),
    ("bf16", 32, 16, 103, 5, (64, 65)),
    ("fp32", 16, 16, 128, 4, (102, 103)),            # 512 heads: eight wavefronts
    ("fp32", 32, 16, 65, 4, (41, 42)),               # 260 heads: by length from 41 on
])
def test_lines_of_the_near_form(dtype, d, b, rows, H, lengths):
    for L in lengths:
        w = with_shape(WORKLOADS["cfg2"], name=f"near-line-{dtype}-d{d}-b{b}-L{L}", B=rows, H=H, L=L, d=d, block=b, window=8, dtype=dtype,
                       qkv_scaled=(dtype == "bf16"), len_lo=1, len_hi=L, stis_block=1, backward=True, seed=7300 + d + L)
        x = make_inputs(w)
        x.valid_len[:4] = [L, 0, 1, L]
        run_case(w, x=x, gate_scale=0.4)


@pytest.mark.parametrize("L", [49, 50, 103, 104])
def test_lines_of_the_near_form_per_position(L):   # 516 key/value heads
    positions.test_backward_under_a_per_position_selection("fp32", 129, 8, 4, L, 8, 32, 16, 16, 4, 8, 1, 1, lengths=((0, L), (1, 1), (128, L)))
