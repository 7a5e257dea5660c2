"""The longest small heads whose backward holds a head in LDS, and one position more: the near form's kernels hold as long ones as the
general kernels do.  Which it is shows in the launches of a captured call: one kernel and the closing of the gate sums, or the streamed
form's two and that."""
import ctypes

import pytest
import torch

from paper_2512_13368_amd import binding as B
from paper_2512_13368_amd.inputs import WORKLOADS, make_inputs, with_shape
from gpu_util import Dev, params
from test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


def _launches(call):
    """Kernel launches of a captured call."""
    call()
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(keep_graph=True), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        call()
    count = ctypes.c_size_t()
    nodes = ctypes.CDLL("libamdhip64.so").hipGraphGetNodes
    nodes.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
    assert nodes(graph.raw_cuda_graph(), None, ctypes.byref(count)) == 0
    return count.value


@pytest.mark.parametrize("mask_block", [1, 2])   # the near form, the general one
@pytest.mark.parametrize("dtype,d,b,L", [
    ("fp32", 8, 16, 496), ("fp32", 16, 16, 240), ("fp32", 16, 8, 240), ("fp32", 32, 16, 240),
    ("bf16", 16, 16, 416), ("bf16", 16, 8, 416), ("bf16", 32, 16, 416), ("bf16", 32, 8, 416),
])
def test_longest_heads_in_lds(dtype, d, b, L, mask_block):
    for length, held in ((L, True), (L + 1, False)):
        w = with_shape(WORKLOADS["cfg2"], name=f"edge-{dtype}-d{d}-b{b}-L{length}-s{mask_block}", B=3, H=2, L=length, d=d, block=b, window=8,
                       dtype=dtype, qkv_scaled=(dtype == "bf16"), len_lo=30, len_hi=length, stis_block=mask_block, seed=993)
        x, sel, f, g = run_case(w, x=make_inputs(w, want_dO=True), backward=True, gate_scale=0.4)
        dv, p = Dev(x), params(w, save_for_bwd=1)
        ws = torch.empty(max(16, B.workspace_bytes(p, B.WS_BWD)), dtype=torch.uint8, device="cuda")
        n = _launches(lambda: B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO, ws=ws, out=g))
        assert n == (2 if held else 3), (length, n)
