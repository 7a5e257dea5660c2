"""Serving mode gives the last block's outputs of a run over all blocks, bit for bit, whatever else is in the batch: on both sides of one
workgroup to a CU (256 of them), with lists and windows of few tiles and of more than 64, with logits that one exponential cannot take."""
import pytest
import torch

from paper_2512_13368_amd import binding as B

pytestmark = pytest.mark.gpu

NAMES = ("O", "o_lt", "o_st", "lse_lt", "lse_st")


def _last_block_alone(rows, H, L, d, b, topk, window, sblk, dtype, amp=1.0):
    """The last block's outputs: of a run over all blocks, of the whole batch in serving mode, of its first two rows in serving mode."""
    print(f"serving bits B{rows} H{H} L{L} d{d} b{b} k{topk} w{window} s{sblk} {dtype} x{amp}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(8100 + L + topk)
    new = lambda *s: torch.randn(s, generator=g, device="cuda")
    Q, K, V = (new(rows, H, L, d).mul_(a).to(dtype) for a in (amp, 1.0, 1.0))
    gw, gb = new(H, 2 * d), new(H)
    vl = torch.randint(1, L + 1, (rows,), generator=g, device="cuda", dtype=torch.int32)
    vl[0], vl[1] = L, L - 2 * b - 6
    lo = (L - 1) // b * b

    def run(n, last):
        p = B.Params(n, H, L, d, b, topk, window, B.F32 if dtype == torch.float32 else B.BF16, stis_mode=int(sblk > 0), stis_block=sblk,
                     save_for_bwd=1, last_block_only=last)
        sel = B.select_blocks(p, Q[:n], K[:n], vl[:n])
        f = B.attn_fwd(p, Q[:n], K[:n], V[:n], vl[:n], sel, gw, gb)
        torch.cuda.synchronize()
        return {name: getattr(f, name)[:, :, lo:].clone() for name in NAMES}

    full, served, few = run(rows, 0), run(rows, 1), run(2, 1)
    for name in NAMES:
        assert bool(full[name].isfinite().all()), name
        assert torch.equal(served[name], full[name]), name
        assert torch.equal(few[name], full[name][:2]), name


@pytest.mark.parametrize("rows,H", [(64, 4), (257, 1)])
@pytest.mark.parametrize("L,topk,window,sblk,amp", [
    (32 * 17, 4, 64, 0, 1.0),
    (32 * 40 + 5, 16, 128, 0, 1.0),
    (32 * 70 + 9, 66, 2200, 0, 1.0),
    (32 * 21 + 30, 12, 100, 32, 1.0),   # all of Eq. 15
    (32 * 22 + 28, 9, 100, 1, 64.0),
])
def test_serving_at_block_32(rows, H, L, topk, window, sblk, amp):
    _last_block_alone(rows, H, L, 64, 32, topk, window, sblk, torch.bfloat16, amp)


@pytest.mark.parametrize("rows,H", [(64, 4), (257, 1)])
@pytest.mark.parametrize("L,topk,window,sblk,amp", [
    (64 * 8, 8, 64, 0, 1.0),
    (64 * 20 + 5, 16, 128, 0, 1.0),
    (64 * 70 + 9, 66, 4400, 0, 1.0),
    (64 * 11 + 60, 10, 100, 64, 1.0),   # all of Eq. 15
    (64 * 12 + 28, 9, 100, 1, 64.0),
])
def test_serving_at_block_64(rows, H, L, topk, window, sblk, amp):
    _last_block_alone(rows, H, L, 64, 64, topk, window, sblk, torch.bfloat16, amp)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("d,b,L,sblk", [
    (8, 16, 200, 1), (8, 8, 1100, 1), (16, 16, 200, 0), (16, 16, 1100, 1), (32, 8, 203, 1), (32, 16, 700, 0),
    (16, 16, 200, 16), (32, 8, 700, 2),
])
def test_serving_of_small_heads(d, b, L, sblk, dtype):
    _last_block_alone(257, 1, L, d, b, 4, 9, sblk, dtype)
