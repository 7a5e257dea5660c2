"""Errors against 64 bits of the small-head kernels' near form: no larger than those of the general kernels, which add the same terms.
The limits are what the general kernels (commit 7a6da87) err by on the same inputs, rounded up in the third place."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import Dev, host, params
from paper_2512_13368_amd import binding as B
from paper_2512_13368_amd.inputs import WORKLOADS, make_inputs, with_shape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,b,L,rows,sblk,limits", [
    # a head in LDS
    ("fp32", 8, 16, 200, 12, 1, {"O": 1.02e-7, "dQ": 1.87e-7, "dK": 2.18e-7, "dV": 1.85e-7}),
    ("fp32", 16, 16, 200, 12, 0, {"O": 1.21e-7, "dQ": 2.25e-7, "dK": 2.71e-7, "dV": 2.42e-7}),
    ("fp32", 32, 16, 200, 12, 0, {"O": 1.35e-7, "dQ": 2.43e-7, "dK": 2.98e-7, "dV": 2.53e-7}),
    ("bf16", 32, 8, 200, 12, 1, {"o_st": 8.25e-8}),
    # streamed
    ("fp32", 8, 16, 1500, 3, 0, {"O": 1.12e-7, "dQ": 2.05e-7, "dK": 2.25e-7, "dV": 2.00e-7}),
    ("fp32", 16, 16, 1500, 3, 0, {"O": 1.33e-7, "dQ": 2.45e-7, "dK": 2.82e-7, "dV": 2.57e-7}),
    ("fp32", 16, 16, 1500, 3, 1, {"O": 1.43e-7, "dQ": 2.43e-7, "dK": 2.88e-7, "dV": 2.66e-7}),
    ("fp32", 32, 16, 1500, 3, 0, {"O": 1.52e-7, "dQ": 2.65e-7, "dK": 3.04e-7, "dV": 2.75e-7}),
    ("bf16", 32, 16, 1500, 3, 1, {"o_st": 9.20e-8}),
    ("bf16", 32, 8, 1500, 3, 1, {"o_st": 9.10e-8}),
])
def test_errors_no_larger_than_the_general_kernels(dtype, d, b, L, rows, sblk, limits):
    w = with_shape(WORKLOADS["cfg2"], name=f"{dtype} d{d} b{b} s{sblk} L{L}", B=rows, H=4, L=L, d=d, block=b, topk=4, window=8, dtype=dtype,
                   len_lo=L // 10, len_hi=L, stis_block=sblk, seed=4100 + d + L + b)
    x = make_inputs(w, want_dO=True)
    x.gate_w = (np.random.default_rng(L + d).standard_normal(x.gate_w.shape) * 0.2).astype(np.float32)
    dv, p = Dev(x), params(w, save_for_bwd=1)
    sel = B.select_blocks(p, dv.Q, dv.K, dv.vl)
    f = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb)
    g = B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO)
    torch.cuda.synchronize()
    args = (x.Q, x.K, x.V, x.valid_len, sel.cpu().numpy(), x.gate_w, x.gate_b)
    refs = (oracle.attn_fwd(*args, b, 4, 8, stis_block=sblk), oracle.attn_bwd(*args, x.dO, b, 4, 8, stis_block=sblk))
    err = {}
    for name in limits:
        got, ref = (getattr(t[name[0] == "d"], name) for t in ((f, g), refs))
        err[name] = float(np.linalg.norm(host(got).reshape(ref.shape) - ref) / np.linalg.norm(ref))
    print(w.name, err, flush=True)
    assert all(err[name] < limits[name] for name in limits), err
