"""Block selection on the GPU against the CPU oracle where its kernels change hands: pairs up to 32 blocks, rows with one
or two candidates per lane up to 128, more than 128; one workgroup per head or pooling and scoring apart, with few
and many heads.  Inputs of small whole numbers make many scores equal, so that the order of equal scores counts too."""
import numpy as np
import pytest
import torch

import oracle
from paper_2512_13368_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,H,L,d,b,k,dtype,stis,last", [
    (3, 2, 9, 8, 8, 2, "fp32", 0, False),         # two blocks, the second of one item
    (3, 2, 512, 16, 16, 5, "fp32", 0, False),     # 32 blocks: the most that pairs take
    (3, 2, 513, 16, 16, 5, "bf16", 0, False),     # 33, few heads: pooling apart, four rows per workgroup
    (50, 4, 513, 8, 16, 4, "fp32", 0, False),     # 33, many heads: one workgroup per head
    (50, 4, 1037, 16, 16, 6, "bf16", 2, False),   # 65 in the bidirectional form: two candidates per lane
    (50, 4, 1024, 8, 8, 7, "fp32", 0, False),     # 128
    (3, 2, 1024, 32, 8, 130, "bf16", 2, False),   # 128, everything selected, padding behind
    (2, 2, 1025, 8, 8, 4, "fp32", 0, False),      # 129
    (70, 4, 4100, 64, 64, 8, "bf16", 0, False),   # pooling apart, sixteen rows per workgroup, ragged last block
    (4, 2, 2040, 64, 32, 8, "bf16", 0, True),     # the last block alone
    (50, 4, 1037, 16, 16, 4, "bf16", 2, False),   # few picks, two candidates per lane, the own block among them
    (3, 2, 2040, 64, 32, 3, "bf16", 0, True),     # few picks for the last block alone
    (3, 2, 1000, 8, 8, 1, "fp32", 0, False),      # nothing to pick beside the own block
    (50, 4, 1037, 16, 16, 6, "fp32", 0, False),   # five passes: the most ...
    (50, 4, 1037, 16, 16, 7, "fp32", 0, False),   # ... six: the search
    (50, 4, 1037, 16, 16, 5, "bf16", 2, False),   # five in the bidirectional form
    (3, 2, 4128, 64, 32, 5, "bf16", 0, True),     # 129 blocks: a thread per candidate, for the last block ...
    (3, 2, 2048, 64, 32, 5, "bf16", 0, True),     # 64 blocks, the last one alone: rows of means ...
    (3, 2, 2049, 64, 32, 5, "bf16", 0, True),     # ... 65: a thread per candidate
    (3, 2, 3088, 16, 16, 200, "bf16", 2, False),  # ... and for every one, 193 of them, all taken
    (3, 2, 8243, 8, 8, 6, "fp32", 0, False),      # 1031 blocks: more than a workgroup has threads
])
def test_selection_at_the_limits_of_its_kernels(rows, H, L, d, b, k, dtype, stis, last):
    rng = np.random.default_rng(L + k)
    Q, K = (rng.integers(-1, 2, size=(rows, H, L, d)).astype(np.float32) for _ in range(2))
    vl = rng.integers(0, L + 1, size=rows).astype(np.int32)
    vl[:2] = [L, max(1, L - b - 3)]
    vl[-1] = 0 if rows > 2 else 1
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    p = B.Params(rows, H, L, d, b, k, 8, B.BF16 if dtype == "bf16" else B.F32, stis_mode=stis, stis_block=b if stis else 0,
                 last_block_only=int(last))
    print(f"select B{rows} H{H} L{L} d{d} b{b} k{k} {dtype} stis{stis} last{last}", flush=True)
    dev = [torch.from_numpy(t).cuda() for t in (Q, K, vl)]
    sel = B.select_blocks(p, dev[0].to(dt), dev[1].to(dt), dev[2]).cpu().numpy()
    want = oracle.select_blocks(Q, K, vl, b, k, bidir=stis == 2)
    if last:
        sel, want = sel[:, :, -1], want[:, :, -1]
    np.testing.assert_array_equal(sel, want)


@pytest.mark.parametrize("dtype,rows,H,L,b,k", [("bf16", 17, 8, 6413, 64, 12), ("fp32", 21, 4, 5003, 32, 9)])
def test_last_block_of_many_keys(dtype, rows, H, L, b, k):
    # 106 and 102 MB of keys, which the last block's selection reads past the caches: the row that the selection of every block has
    rng = np.random.default_rng(L)
    Q, K = (rng.integers(-2, 3, size=(rows, H, L, 64), dtype=np.int8).astype(np.float32) for _ in range(2))
    vl = rng.integers(1, L + 1, size=rows).astype(np.int32)
    vl[:3] = [L, L - b - 3, 1]
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Qd, Kd, vld = torch.from_numpy(Q).cuda().to(dt), torch.from_numpy(K).cuda().to(dt), torch.from_numpy(vl).cuda()
    assert Kd.numel() * Kd.element_size() > 100 << 20

    def last_row(**kw):
        p = B.Params(rows, H, L, 64, b, k, 8, B.BF16 if dtype == "bf16" else B.F32, **kw)
        return B.select_blocks(p, Qd, Kd, vld)[:, :, -1].cpu().numpy()

    last = last_row(last_block_only=1)
    np.testing.assert_array_equal(last, last_row())
    pairs = np.array([0, H + 1, 2 * H, rows * H - 1], np.int32)
    want = oracle.select_blocks(Q, K, vl, b, k, bh_list=pairs)[:, :, -1]
    np.testing.assert_array_equal(last.reshape(-1, k)[pairs], want.reshape(-1, k)[pairs])


@pytest.mark.parametrize("L,d,b,k,last", [
    (2632, 64, 64, 9, False), (2576, 64, 64, 9, True),   # 8 rows left over; 16, a quarter of a block
    (2577, 64, 64, 9, False), (2609, 64, 64, 9, True),   # 17, 49: a wavefront with that block sums all of its blocks row by row
    (2600, 64, 32, 9, False), (2601, 64, 32, 9, True),   # 8, a quarter; 9
    (2591, 32, 32, 9, False), (2560, 32, 32, 9, False),  # 31; none
    (5150, 16, 64, 9, False), (5151, 8, 64, 9, False),   # a wavefront with many blocks, 30 and 31 rows left over
])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_pooling_beside_a_ragged_block(L, d, b, k, last, dtype):
    # whole blocks are pooled by a loop of their own, histories that start inside a block leave another ragged one at the front
    rng = np.random.default_rng(L + d)
    Q, K = (rng.integers(-2, 3, size=(3, 4, L, d)).astype(np.float32) for _ in range(2))
    vl = np.array([L, L - b - 3, L // 2 + 5], np.int32)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    p = B.Params(3, 4, L, d, b, k, 8, B.BF16 if dtype == "bf16" else B.F32, last_block_only=int(last))
    dev = [torch.from_numpy(t).cuda() for t in (Q, K, vl)]
    sel = B.select_blocks(p, dev[0].to(dt), dev[1].to(dt), dev[2]).cpu().numpy()
    want = oracle.select_blocks(Q, K, vl, b, k)
    if last:
        sel, want = sel[:, :, -1], want[:, :, -1]
    np.testing.assert_array_equal(sel, want)
