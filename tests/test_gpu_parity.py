"""GPU parity: the HIP path behind the C ABI against the CPU oracle on the same seeded inputs.

Block selection must match bit-exactly; outputs and gradients within
|x-ref| <= tol*(|ref| + rms(ref)), tol = 1e-4 (fp32) or 2e-2 (bf16 storage, fp32 accumulate).
Small cases compare every element; the full-size workloads compare all selections and the
outputs of sampled (row, head) pairs the oracle can afford.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import TOL, Dev, assert_close, host, params, pick_pairs
from paper_2512_13368_amd import binding as B
from paper_2512_13368_amd.inputs import WORKLOADS, make_inputs, with_shape

pytestmark = pytest.mark.gpu


def run_case(w, x=None, pairs=None, backward=None, check_dense=False, gate_scale=None, branches_coincide=False,
             scale=None, sel_edit=None):
    if x is None:
        x = make_inputs(w, want_dO=True)
    if gate_scale is not None:  # stronger gate weights exercise the gate path beyond alpha ~ 0.5
        rng = np.random.default_rng(w.seed + 7)
        x.gate_w = (rng.standard_normal(x.gate_w.shape) * gate_scale).astype(np.float32)
        x.gate_b = (rng.standard_normal(x.gate_b.shape) * 0.5).astype(np.float32)
    backward = w.backward if backward is None else backward
    tol = TOL[w.dtype]
    print(f"case {w.name} B{w.B} H{w.H} L{w.L} d{w.d} b{w.block} k{w.topk} w{w.window} {w.dtype} "
          f"bwd={backward}", flush=True)
    dv = Dev(x)
    sc = {} if scale is None else dict(softmax_scale=scale)   # None: the default 1/sqrt(d) on both sides
    p = params(w, save_for_bwd=1, **sc)
    sel = B.select_blocks(p, dv.Q, dv.K, dv.vl)
    torch.cuda.synchronize()

    # --- selection: every (row, head), bit-exact ---
    sel_ref = oracle.select_blocks(x.Q, x.K, x.valid_len, w.block, w.topk, bidir=w.bidir)
    np.testing.assert_array_equal(sel.cpu().numpy(), sel_ref)
    if sel_edit is not None:  # a caller-built selection: both sides get the same edited rows
        sel_ref = np.ascontiguousarray(sel_edit(sel_ref.copy()), dtype=np.int32)
        sel = torch.from_numpy(sel_ref).cuda()

    f = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb)
    g = B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO) if backward else None
    torch.cuda.synchronize()

    # --- outputs: listed pairs ---
    bh = None if pairs is None else np.asarray(pairs, np.int32)
    take = (lambda t: host(t).reshape(w.B * w.H, *t.shape[2:])[bh if bh is not None else slice(None)])
    fr = oracle.attn_fwd(x.Q, x.K, x.V, x.valid_len, sel_ref, x.gate_w, x.gate_b, w.block, w.topk,
                         w.window, scale=scale, bh_list=bh, stis_block=w.stis_block, bidir=w.bidir)
    assert_close(take(f.o_lt), fr.o_lt, tol, "o_lt")
    assert_close(take(f.o_st), fr.o_st, tol, "o_st")
    assert_close(take(f.O), fr.O, tol, "O")
    assert_close(take(f.lse_lt), fr.lse_lt, tol, "lse_lt")
    assert_close(take(f.lse_st), fr.lse_st, tol, "lse_st")
    # pad rows are exactly zero
    for r in range(w.B):
        p0 = w.L - int(x.valid_len[r])
        if p0 > 0:
            assert float(f.O[r, :, :p0].abs().max()) == 0.0
            assert float(f.o_lt[r, :, :p0].abs().max()) == 0.0 and float(f.o_st[r, :, :p0].abs().max()) == 0.0

    # forward without the saved tensors gives the same O
    p0_ = params(w, save_for_bwd=0, **sc)
    f2 = B.attn_fwd(p0_, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb)
    assert torch.equal(f2.O, f.O)

    if backward:
        gr = oracle.attn_bwd(x.Q, x.K, x.V, x.valid_len, sel_ref, x.gate_w, x.gate_b, x.dO, w.block,
                             w.topk, w.window, scale=scale, bh_list=bh, stis_block=w.stis_block, bidir=w.bidir)
        assert_close(take(g.dQ), gr.dQ, tol, "dQ")
        assert_close(take(g.dK), gr.dK, tol, "dK")
        assert_close(take(g.dV), gr.dV, tol, "dV")
        if bh is None and not branches_coincide:  # gate gradients sum over every pair
            assert_close(host(g.d_gate_w), gr.d_gate_w, tol, "d_gate_w")
            assert_close(host(g.d_gate_b), gr.d_gate_b, tol, "d_gate_b")
        assert bh is None or not w.backward, "a workload whose outputs include the gate gradients runs every pair"
        if branches_coincide:
            # o_lt == o_st in exact arithmetic: the gate gradients are exactly zero there, so the
            # relative criterion has nothing to hold on to; the kernels' two branches round
            # differently, which leaves sums of products of rounding errors
            assert float(np.abs(gr.d_gate_w).max()) == 0.0 and float(np.abs(gr.d_gate_b).max()) == 0.0
            assert float(g.d_gate_w.abs().max()) < 1e-3 * tol and float(g.d_gate_b.abs().max()) < 1e-3 * tol
        for r in range(w.B):
            p0 = w.L - int(x.valid_len[r])
            if p0 > 0:
                for t in (g.dQ, g.dK, g.dV):
                    assert float(t[r, :, :p0].abs().max()) == 0.0
        # determinism: a second run is bitwise identical
        g2 = B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO)
        for a, b_ in ((g.dQ, g2.dQ), (g.dK, g2.dK), (g.dV, g2.dV), (g.d_gate_w, g2.d_gate_w),
                      (g.d_gate_b, g2.d_gate_b)):
            assert torch.equal(a, b_)

    if check_dense:
        lse = torch.empty((w.B, w.H, w.L), dtype=torch.float32, device="cuda")
        Od, _ = B.dense_causal_fwd(p, dv.Q, dv.K, dv.V, dv.vl, lse=lse)
        torch.cuda.synchronize()
        Or, lr = oracle.dense_causal_fwd(x.Q, x.K, x.V, x.valid_len, scale=scale, bh_list=bh)
        assert_close(take(Od), Or, tol, "dense O")
        assert_close(take(lse), lr, tol, "dense lse")
    return x, sel, f, g


def test_cfg1_all_elements():
    run_case(WORKLOADS["cfg1"], backward=True, check_dense=True)
    run_case(WORKLOADS["cfg1"], backward=True, gate_scale=0.5)


def test_cfg2_all_elements():
    run_case(WORKLOADS["cfg2"], backward=True, check_dense=True)


def test_cfg3_reduced_all_elements():
    run_case(with_shape(WORKLOADS["cfg3"], B=6), backward=True, check_dense=True, gate_scale=0.3)


def test_cfg3_full_size_sampled():
    w = WORKLOADS["cfg3"]
    run_case(w, pairs=pick_pairs(w, 12), backward=True)


def test_cfg4_reduced_all_elements():
    # several query blocks per head with the real block/top-k/window, small enough for every element
    run_case(with_shape(WORKLOADS["cfg4"], B=2, H=2, L=1536, len_lo=700, len_hi=1536), backward=True,
             check_dense=True)


def test_cfg4_full_size_sampled():
    # The launch configuration the benchmark times (plain causal window, every query block), forward
    # and backward.  The kernels deal (row, head) pairs to the eight XCDs in contiguous ranges of 16:
    # two pairs of every range are compared (first and last pair of the workload among them).
    w = WORKLOADS["cfg4"]
    total = w.B * w.H
    pairs = sorted({int(t) for t in np.linspace(0, total - 1, 16).round()})
    assert len(pairs) == 16 and all(sum(1 for q in pairs if q // 16 == r) == 2 for r in range(8))
    run_case(w, pairs=pairs, backward=True)


def test_cfg4_full_size_sampled_full_short_term_mask():
    # cfg4 at full size with all of Eq. 15 (mask block = tile): seven more key blocks per query block
    w = with_shape(WORKLOADS["cfg4"], name="cfg4-eq15", stis_block=64)
    run_case(w, pairs=pick_pairs(w, 2), backward=True)


def test_cfg4_full_size_sampled_paper_mask_block():
    # cfg4 at full size with all of Eq. 15 and the paper's mask block 1 (matrix-core kernels, mask block below the tile)
    w = with_shape(WORKLOADS["cfg4"], name="cfg4-eq15-blk1", stis_block=1, window=8)
    run_case(w, pairs=pick_pairs(w, 2), backward=True)


def test_cfg5_full_size_every_pair():
    # the training-step workload at full size, every (row, head) pair: dQ, dK, dV element by element and
    # the gate gradients, whose two-level reduction runs with its full chunk and slice counts only here
    run_case(WORKLOADS["cfg5"], backward=True)


@pytest.mark.parametrize("dtype,d,b", [("fp32", 32, 8), ("fp32", 64, 16), ("bf16", 32, 32), ("bf16", 64, 8),
                                       ("fp32", 64, 64), ("bf16", 32, 64), ("fp32", 32, 32), ("bf16", 64, 16),
                                       ("bf16", 64, 32), ("bf16", 64, 64)])
def test_shape_matrix(dtype, d, b):
    # ragged tail (L not a multiple of b), mixed lengths, every supported (dtype, d, b)
    L = 3 * b + b // 2 + 1
    w = with_shape(WORKLOADS["cfg1"], name=f"m-{dtype}-{d}-{b}", B=3, H=2, L=L, d=d, block=b, topk=3,
                   window=b + 3, dtype=dtype, len_lo=1, len_hi=L, qkv_scaled=(dtype == "bf16"), seed=200 + d + b)
    x = make_inputs(w, want_dO=True)
    # a full row (the two branches differ), a row starting inside a block, a row shorter than a block
    x.valid_len[:] = [L, L - b - 3, b // 2 + 1]
    run_case(w, x=x, backward=True, check_dense=True, gate_scale=0.4)


@pytest.mark.parametrize("name,shape", [
    ("cfg1", dict(topk=4)),                                                                  # fp32 matrix instructions, fp32
    ("cfg2", dict(B=4, dtype="bf16", qkv_scaled=True)),                                      # fp32 matrix instructions, bf16
    ("cfg1", dict(topk=4, d=64)),                                                            # scalar kernels, fp32
    ("cfg2", dict(B=4, d=64, dtype="bf16", qkv_scaled=True)),                                # scalar kernels, bf16
    ("cfg3", dict(B=3, L=32 * 9 + 11, len_lo=40, len_hi=32 * 9 + 11, topk=5)),               # matrix cores, b = 32
    ("cfg4", dict(B=2, H=2, L=64 * 9, len_lo=300, len_hi=64 * 9, topk=6)),                   # matrix cores, b = 64
    ("cfg4", dict(B=1, H=2, L=64 * 70, len_lo=64 * 70, len_hi=64 * 70, topk=67, window=64)),  # a row read in two chunks
])
def test_selection_rows_with_holes(name, shape):
    # A caller-built selection row may hold entries outside [0, NB) anywhere: every kernel family skips
    # them where they stand (as the oracle's mask does) in forward, dQ and dK/dV alike.
    w = with_shape(WORKLOADS[name], name=name + "-holes", **shape)

    def punch(sel):
        NB = sel.shape[2]
        rng = np.random.default_rng(w.seed + 13)
        for r in range(sel.shape[0]):
            for h in range(sel.shape[1]):
                for I in range(NB):
                    row = sel[r, h, I]
                    cnt = int((row >= 0).sum())
                    if cnt < 3:
                        continue
                    kind = int(rng.integers(0, 4))
                    if kind == 0:
                        row[int(rng.integers(1, cnt - 1))] = -1            # a hole inside the list
                    elif kind == 1:
                        row[0] = NB + 3                                    # an id past the last block, up front
                    elif kind == 2:
                        row[0] = -1
                        row[cnt - 2] = -5                                  # two holes
                    # kind 3: the row stays as selected
                    own = np.where(row == I)[0]
                    assert own.size == 1                                   # the query's own block is still listed
        return sel

    run_case(w, backward=True, gate_scale=0.4, sel_edit=punch)


@pytest.mark.parametrize("b", [32, 64])
def test_a_hole_in_front_of_the_own_block(b):
    # the first block with a valid query (padding before it) lists an entry that is no block, then itself
    L = 5 * b
    w = with_shape(WORKLOADS["cfg4"], name=f"hole-in-front-{b}", B=2, H=2, L=L, block=b, topk=3, window=b, len_lo=1, len_hi=L, seed=640 + b)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:] = [L - b - 5, 2 * b + 9]

    def shift(sel):
        for r, first in ((0, 1), (1, 2)):
            sel[r, :, first] = [-1, first, -1]
        return sel

    run_case(w, x=x, backward=True, gate_scale=0.4, sel_edit=shift)


@pytest.mark.parametrize("name,shape", [
    ("cfg1", dict(topk=4)),                                                                    # fp32 matrix instructions, fp32
    ("cfg2", dict(B=3, dtype="bf16", qkv_scaled=True)),                                        # fp32 matrix instructions, bf16
    ("cfg1", dict(topk=4, d=64)),                                                              # scalar kernels
    ("cfg3", dict(B=3, L=32 * 9 + 11, len_lo=40, len_hi=32 * 9 + 11, topk=5)),                 # matrix cores, b = 32
    ("cfg3", dict(B=3, L=32 * 9, len_lo=40, len_hi=32 * 9, topk=5, stis_block=32)),            # ... with all of Eq. 15
    ("cfg4", dict(B=3, H=2, L=64 * 7 + 20, len_lo=200, len_hi=64 * 7 + 20, topk=6)),           # matrix cores, b = 64
    ("cfg4", dict(B=3, H=2, L=64 * 7, len_lo=200, len_hi=64 * 7, topk=6, stis_block=1)),       # ... with all of Eq. 15
])
def test_selection_rows_that_name_later_blocks(name, shape):
    # caller-built rows list blocks after the query block: they contribute nothing, in forward and backward alike
    w = with_shape(WORKLOADS[name], name=name + "-later", **shape)

    def later(sel):
        NB = sel.shape[2]
        for I in range(NB):
            for r in range(sel.shape[0]):
                for h in range(sel.shape[1]):
                    row = sel[r, h, I]
                    others = [e for e in range(w.topk) if row[e] != I]
                    if (row == I).any():
                        for e, J in zip(others[(I + r) % 2:], dict.fromkeys([min(I + 1, NB - 1), NB - 1])):
                            if J > I:
                                row[e] = J
        return sel

    run_case(w, backward=True, gate_scale=0.4, sel_edit=later)


@pytest.mark.parametrize("b,stis_block,topk", [(32, 0, 3), (32, 32, 3), (32, 8, 2), (64, 0, 3), (64, 64, 3), (64, 1, 2)])
def test_blocks_of_padding_may_hold_anything(b, stis_block, topk):
    # the matrix-core kernels, which multiply whole blocks: those of nothing but padding hold NaN, also where a caller-built row names
    # one of them, or an entry that is no block
    L = 6 * b + 9
    w = with_shape(WORKLOADS["cfg4"], name=f"padding-{b}-{stis_block}", B=4, H=2, L=L, block=b, topk=topk, window=b + 3, len_lo=1,
                   len_hi=L, stis_block=stis_block, seed=680 + b + stis_block)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:] = [L - 1, L - b - b // 2, 3 * b + 5, 4]
    first = (L - x.valid_len) // b
    for r in range(w.B):
        for t in (x.Q, x.K, x.V, x.dO):
            t[r, :, : first[r] * b] = np.nan

    def padding_named(sel):
        for r in range(w.B):
            for I in range(first[r], w.NB):
                e = next(e for e in range(topk) if sel[r, 0, I, e] != I)
                sel[r, 0, I, e] = 0 if first[r] > 0 else -1      # a block of padding, if the row has one
                if I % 2:
                    sel[r, 1, I, e] = -1
        return sel

    run_case(w, x=x, backward=True, gate_scale=0.4, check_dense=True, sel_edit=padding_named)


@pytest.mark.parametrize("b,stis_block,topk", [(32, 0, 3), (32, 32, 3), (32, 8, 2), (64, 0, 3), (64, 64, 3), (64, 1, 2)])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_padding_of_a_partly_valid_block_may_hold_any_finite_value(b, stis_block, topk, sign):
    # the matrix-core kernels: the largest there is in all four tensors, whose products overflow
    L = 6 * b + 9
    w = with_shape(WORKLOADS["cfg4"], name=f"large-padding-{b}-{stis_block}", B=4, H=2, L=L, block=b, topk=topk, window=b + 3, len_lo=1,
                   len_hi=L, stis_block=stis_block, seed=690 + b + stis_block)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:] = [L - 1, L - b - b // 2, 3 * b + 5, 4]  # (of a block of 64 also one whose first half is padding)
    for r in range(w.B):
        for t in (x.Q, x.K, x.V, x.dO):
            t[r, :, : L - x.valid_len[r]] = sign * torch.finfo(torch.bfloat16).max
    run_case(w, x=x, backward=True, gate_scale=0.4, check_dense=True)


@pytest.mark.parametrize("b", [32, 64])
def test_a_gate_that_shuts_a_branch(b):
    # one head's gate closes the long-term branch, the other's the short-term one (a weight of zero, whose logarithm goes into no
    # exponent); dO in the padding of a partly valid block is the largest there is, and its products overflow
    L = 4 * b + 9
    w = with_shape(WORKLOADS["cfg4"], name=f"shut-{b}", B=2, H=2, L=L, block=b, topk=2, window=b + 3, len_lo=1, len_hi=L, backward=False,
                   seed=670 + b)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:] = [L - b // 2, b + 5]
    x.gate_b[:] = [-200.0, 200.0]
    for r in range(w.B):
        x.dO[r, :, : L - int(x.valid_len[r])] = torch.finfo(torch.bfloat16).max
    run_case(w, x=x, backward=True, pairs=range(4))  # (all of them; the gate's own gradients are zero in fp32, e^-200 in exact arithmetic)


@pytest.mark.parametrize("b,topk,window", [(64, 1, 5), (64, 2, 40), (32, 1, 200), (32, 2, 7), (64, 3, 20)])
def test_matrix_core_few_key_rows(b, topk, window):
    # bf16 d=64 (the matrix-core kernels) where rows see only a few keys far beyond the first blocks:
    # top-k of one or two (every query block's long-term rows may have few keys), windows shorter than
    # 32 (every short-term row has few keys).  Exercises the two-term operands and the residual passes of
    # the backward kernels on most tiles, and the inverse list's few-keys flag.
    L = 5 * b + b // 2 + 3
    w = with_shape(WORKLOADS["cfg4"], name=f"few-{b}-{topk}-{window}", B=3, H=2, L=L, d=64, block=b, topk=topk,
                   window=window, len_lo=1, len_hi=L, seed=500 + b + topk + window)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:] = [L, L - b - 5, 2 * b + 1]
    run_case(w, x=x, backward=True, check_dense=True, gate_scale=0.4)


def test_matrix_core_long_walks():
    # bf16 d=64 b=32 with more than a hundred tiles per query block.  First a window wider than the
    # sequence plus a top-k that keeps every block: both branches are dense causal attention (forward;
    # in that limit the gradient rms is set by thousands of late rows with tiny gradients, which makes
    # the rms-floored tolerance a 5-sigma test for the first rows, so backward is checked on the second
    # case).  Then window tiles and selected tiles each above 64 entries: the selection row is read in
    # two chunks, and the walk is longer than any of the workloads'.
    L = 32 * 104 + 5
    w = with_shape(WORKLOADS["cfg3"], name="long-dense-limit", B=1, H=2, L=L, d=64, block=32, topk=105,
                   window=L, len_lo=L, len_hi=L, seed=611)
    x2, sel, f, _ = run_case(w, x=make_inputs(w, want_dO=True), backward=False, check_dense=True, gate_scale=0.4)
    dv = Dev(x2)
    Od, _ = B.dense_causal_fwd(params(w), dv.Q, dv.K, dv.V, dv.vl)
    torch.cuda.synchronize()
    assert_close(host(f.o_lt), host(Od), 2e-2, "o_lt vs dense kernel")
    assert_close(host(f.o_st), host(Od), 2e-2, "o_st vs dense kernel")
    w = with_shape(WORKLOADS["cfg3"], name="long-mixed", B=2, H=1, L=L, d=64, block=32, topk=70,
                   window=32 * 66, len_lo=L - 700, len_hi=L, seed=612)
    run_case(w, backward=True, gate_scale=0.4)


def test_seeded_random_shapes():
    # Sixty seeded draws of (dtype, d, b, L, k, w, lengths) over everything the library accepts: odd
    # lengths, rows that start in the middle of a block, top-k from 1 to beyond the number of blocks,
    # windows from 1 to beyond L.  The bf16 matrix-core kernels get half of the draws, the scalar ones (d = 64, or blocks from
    # 32) and the fp32 matrix instructions (d = 32, block 8 or 16) the others.
    rng = np.random.default_rng(4242)
    for case in range(60):
        mfma = case % 2 == 0
        dtype = "bf16" if mfma or rng.random() < 0.3 else "fp32"
        d = 64 if mfma else int(rng.choice([32, 64]))
        b = int(rng.choice([32, 64])) if mfma else int(rng.choice([8, 16, 32, 64]))
        nb = int(rng.integers(1, 13))
        L = max(2, nb * b - int(rng.integers(0, b)))  # (one key per row would make dQ, dK identically zero)
        topk = int(rng.choice([1, 2, 3, nb, nb + 3]))
        window = int(rng.choice([1, 2, b - 1, b, b + 1, 2 * b + 5, L, L + 7]))
        sblk = int(rng.choice([0, 0, b, 1, 3, 2 * b]))  # a third of the draws use all of Eq. 15
        w = with_shape(WORKLOADS["cfg1"], name=f"rnd{case}", B=4, H=2, L=L, d=d, block=b, topk=max(1, topk),
                       window=max(1, window), dtype=dtype, len_lo=0, len_hi=L, qkv_scaled=(dtype == "bf16"),
                       seed=7000 + case, stis_block=sblk)
        x = make_inputs(w, want_dO=True)
        x.valid_len[:] = [L, int(rng.integers(0, L + 1)), int(rng.integers(0, L + 1)), min(L, 1 + int(rng.integers(0, b)))]
        same = w.topk >= w.NB and (w.window >= L or sblk >= L)  # both branches are dense causal attention
        run_case(w, x=x, backward=True, check_dense=(case % 4 == 0), gate_scale=0.4, branches_coincide=same)


@pytest.mark.parametrize("dtype,d,b,sblk,window,L", [
    ("fp32", 32, 8, 1, 8, 200),      # the paper's own setting: mask block 1, window 8
    ("fp32", 64, 16, 4, 6, 131),     # mask blocks smaller than the tiles, ragged tail
    ("fp32", 32, 16, 16, 20, 150),   # mask block = tile
    ("bf16", 32, 32, 8, 3, 300),
    ("bf16", 64, 16, 64, 5, 333),    # mask blocks larger than the tiles
    ("fp32", 64, 8, 200, 2, 90),     # one mask block: the short-term branch is dense causal attention
    ("bf16", 64, 32, 32, 40, 647),   # the matrix-core kernels: mask block = tile
    ("bf16", 64, 64, 64, 128, 1157),
    ("bf16", 64, 64, 64, 5, 577),    # short window: few-key rows in the band tiles
    ("bf16", 64, 32, 32, 1, 1024),   # no ragged tail: the last block term covers a whole tile
    ("bf16", 64, 64, 32, 70, 700),   # bf16 d=64 with a mask block that is not the tile: scalar kernels
    ("fp32", 32, 16, 4, 1, 131),     # window 1 and a short last block: last-block keys lie below the window tiles
    ("fp32", 8, 16, 3, 2, 100),      # mask block that is no power of two and does not divide the tile
    ("bf16", 16, 64, 1, 8, 1000),    # mask block 1 under a 64-row tile: 10 gathered runs per row
    ("bf16", 64, 64, 1, 8, 1100),    # the matrix-core kernels with a mask block below the tile: the paper's block 1
    ("bf16", 64, 32, 1, 8, 700),
    ("bf16", 64, 64, 8, 3, 577),
    ("bf16", 64, 32, 4, 40, 333),
    ("bf16", 64, 64, 16, 1, 64 * 9),  # window 1, no ragged tail
])
def test_full_short_term_mask(dtype, d, b, sblk, window, L):
    # stis_mode 1: window + whole blocks at power-of-two block distances + last block (Eq. 15, causal)
    w = with_shape(WORKLOADS["cfg1"], name=f"stis-{dtype}-{d}-{b}-{sblk}", B=3, H=2, L=L, d=d, block=b, topk=3,
                   window=window, dtype=dtype, len_lo=1, len_hi=L, qkv_scaled=(dtype == "bf16"), seed=900 + d + b + sblk,
                   stis_block=sblk)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:] = [L, L - b - 3, max(1, L // 3)]
    run_case(w, x=x, backward=True, gate_scale=0.4)


@pytest.mark.parametrize("dtype,d,b,sblk,window,L,topk", [
    ("fp32", 32, 8, 1, 8, 200, 4),       # the paper's mask setting: mask block 1, window 8
    ("fp32", 8, 16, 1, 8, 100, 4),       # ... at its head size
    ("fp32", 64, 16, 4, 6, 131, 3),      # mask blocks smaller than the tiles, ragged tail
    ("fp32", 32, 16, 16, 20, 150, 3),    # mask block = tile
    ("bf16", 32, 32, 8, 3, 300, 2),
    ("bf16", 64, 16, 64, 5, 333, 5),     # mask blocks larger than the tiles
    ("bf16", 64, 32, 32, 40, 647, 4),    # shapes the matrix cores serve in the causal forms: scalar kernels here
    ("bf16", 64, 64, 0, 70, 700, 3),     # mask block 0 = the selection block
    ("fp32", 16, 8, 3, 1, 90, 1),        # window 1, top-k 1 (own block only), mask block that is no power of two
    ("fp32", 32, 8, 200, 2, 90, 20),     # one mask block and every block selected: both branches are full attention
])
def test_bidirectional_form(dtype, d, b, sblk, window, L, topk):
    # stis_mode 2: Eq. 15 as printed (symmetric) and selected blocks seen whole, for bidirectional backbones
    w = with_shape(WORKLOADS["cfg1"], name=f"bidir-{dtype}-{d}-{b}-{sblk}", B=3, H=2, L=L, d=d, block=b, topk=topk,
                   window=window, dtype=dtype, len_lo=1, len_hi=L, qkv_scaled=(dtype == "bf16"), seed=2300 + d + b + sblk,
                   stis_block=sblk, bidir=True)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:] = [L, L - b - 3, max(1, L // 3)]
    same = sblk >= L and topk >= w.NB
    run_case(w, x=x, backward=True, gate_scale=0.4, branches_coincide=same)


def test_bidirectional_serving_mode():
    w = with_shape(WORKLOADS["cfg1"], name="bidir-serve", B=3, H=2, L=77, d=16, block=8, topk=3, window=5, stis_block=2,
                   bidir=True, len_lo=20, len_hi=77)
    x = make_inputs(w)
    dv = Dev(x)
    sel_all = B.select_blocks(params(w), dv.Q, dv.K, dv.vl)
    f_all = B.attn_fwd(params(w), dv.Q, dv.K, dv.V, dv.vl, sel_all, dv.gw, dv.gb)
    sel = torch.full_like(sel_all, -7)
    B.select_blocks(params(w, last_block_only=1), dv.Q, dv.K, dv.vl, sel=sel)
    O = torch.full_like(f_all.O, 3.0)
    B.attn_fwd(params(w, last_block_only=1), dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, out=B.FwdOut(O))
    torch.cuda.synchronize()
    lo = (w.NB - 1) * w.block
    assert torch.equal(sel[:, :, -1], sel_all[:, :, -1]) and torch.equal(O[:, :, lo:], f_all.O[:, :, lo:])
    assert bool((O[:, :, :lo] == 3.0).all())


@pytest.mark.parametrize("name,shape", [
    ("cfg1", dict()),                                                          # fp32 matrix instructions
    ("cfg1", dict(d=64)),                                                      # scalar kernels, fp32
    ("cfg3", dict(B=3, L=32 * 9 + 11, len_lo=40, len_hi=32 * 9 + 11)),          # matrix cores, ragged last block
    ("cfg4", dict(B=2, H=2, L=64 * 6, len_lo=100, len_hi=64 * 6)),              # matrix cores, b = 64
    ("cfg4", dict(B=2, H=2, L=64 * 5 + 3, len_lo=64 * 5 + 3, len_hi=64 * 5 + 3, stis_block=64)),
    ("cfg2", dict(B=5, H=8, d=8, L=197, len_lo=30, len_hi=197, topk=4, window=8, stis_block=1)),  # the paper's setting
])
def test_serving_mode_last_block_only(name, shape):
    # last_block_only: selection row and output rows of the last query block equal the full run's, and
    # nothing else in the buffers is written
    w = with_shape(WORKLOADS[name], name=name + "-serve", **shape)
    x = make_inputs(w)
    dv = Dev(x)
    p_all = params(w)
    p_last = params(w, last_block_only=1)
    sel_all = B.select_blocks(p_all, dv.Q, dv.K, dv.vl)
    f_all = B.attn_fwd(p_all, dv.Q, dv.K, dv.V, dv.vl, sel_all, dv.gw, dv.gb)
    sel = torch.full_like(sel_all, -7)
    B.select_blocks(p_last, dv.Q, dv.K, dv.vl, sel=sel)
    O = torch.full_like(f_all.O, 3.0)
    B.attn_fwd(p_last, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, out=B.FwdOut(O))
    torch.cuda.synchronize()
    lo = (w.NB - 1) * w.block
    assert torch.equal(sel[:, :, -1], sel_all[:, :, -1]) and bool((sel[:, :, :-1] == -7).all())
    assert torch.equal(O[:, :, lo:], f_all.O[:, :, lo:]) and bool((O[:, :, :lo] == 3.0).all())
    # and the last block agrees with the oracle
    sel_ref = oracle.select_blocks(x.Q, x.K, x.valid_len, w.block, w.topk)
    np.testing.assert_array_equal(sel[:, :, -1].cpu().numpy(), sel_ref[:, :, -1])
    fr = oracle.attn_fwd(x.Q, x.K, x.V, x.valid_len, sel_ref, x.gate_w, x.gate_b, w.block, w.topk, w.window,
                         stis_block=w.stis_block)
    assert_close(host(O[:, :, lo:]).reshape(w.B * w.H, w.L - lo, w.d), fr.O[:, lo:], TOL[w.dtype], "O (last block)")
    with pytest.raises(B.BlossomError):  # no backward in serving mode
        f = B.attn_fwd(params(w, save_for_bwd=1), dv.Q, dv.K, dv.V, dv.vl, sel_all, dv.gw, dv.gb)
        B.attn_bwd(params(w, save_for_bwd=1, last_block_only=1), dv.Q, dv.K, dv.V, dv.vl, sel_all, dv.gw, dv.gb, f,
                   torch.zeros_like(f.O))


@pytest.mark.parametrize("b", [32, 64])
def test_matrix_core_sharp_softmax(b):
    # logits eight times the usual spread (queries scaled by a power of two, so they stay bf16 values): block 64, whose softmax
    # keeps a reference, has to move it many times per row (block 32 keeps none: test_gpu_merged_walk.py drives it out of its
    # range); backward sees probabilities close to one everywhere
    L = 9 * b + 5
    w = with_shape(WORKLOADS["cfg3"], name=f"sharp-{b}", B=2, H=2, L=L, d=64, block=b, topk=4, window=b + 9,
                   len_lo=L - 70, len_hi=L, seed=1200 + b)
    x = make_inputs(w, want_dO=True)
    x.Q *= np.float32(8.0)
    run_case(w, x=x, backward=True, check_dense=True, gate_scale=0.4)


def test_selection_ties():
    # equal scores: planted duplicate key blocks (bit-identical scores, the lower index must win), and
    # zero scores from two different causes (a zero key block, and a key block orthogonal to the query sum)
    w = with_shape(WORKLOADS["cfg1"], name="dup", B=2, H=2, L=80, d=32, block=8, topk=3, len_lo=70, len_hi=80, seed=3)
    for dtype in ("fp32", "bf16"):
        wd = with_shape(w, dtype=dtype)
        xd = make_inputs(wd)
        xd.K[:, :, 32:40] = xd.K[:, :, 16:24]
        xd.K[:, :, 48:56] = xd.K[:, :, 16:24]
        xd.K[:, :, 56:64] = xd.K[:, :, 16:24]
        dv = Dev(xd)
        sel = B.select_blocks(params(wd), dv.Q, dv.K, dv.vl)
        np.testing.assert_array_equal(sel.cpu().numpy(), oracle.select_blocks(xd.Q, xd.K, xd.valid_len, 8, 3))
    wz = with_shape(WORKLOADS["cfg1"], name="zeros", B=1, H=1, L=24, d=32, block=8, topk=2, len_lo=24, len_hi=24)
    xz = make_inputs(wz)
    xz.Q[:] = 0.0
    xz.K[:] = 0.0
    xz.Q[0, 0, 16:24, 0] = -1.0
    xz.K[0, 0, 8:16, 1] = 1.0
    sel_ref, sc = oracle.select_blocks(xz.Q, xz.K, xz.valid_len, 8, 2, want_scores=True)
    assert sc[0, 2, 0] == 0.0 and sc[0, 2, 1] == 0.0
    dv = Dev(xz)
    np.testing.assert_array_equal(B.select_blocks(params(wz), dv.Q, dv.K, dv.vl).cpu().numpy(), sel_ref)
    assert [int(t) for t in sel_ref[0, 0, 2]] == [0, 2]


def test_many_blocks_backward():
    # more than 2048 blocks per row: the inverse selection list then runs with one wavefront per (row, head)
    # and its counters no longer fit four-fold in LDS; scalar kernels (more than 16384 positions), fp32
    w = with_shape(WORKLOADS["cfg1"], name="many-blocks", B=1, H=2, L=8 * 2100 + 3, d=32, block=8, topk=4, window=11,
                   len_lo=8 * 2100 - 50, len_hi=8 * 2100 + 3, seed=77)
    run_case(w, backward=True, gate_scale=0.4)


@pytest.mark.parametrize("L", [8 * 488, 8 * 488 + 1])
def test_inverse_lists_beside_the_gate_pass(L):
    # the most blocks whose lists are made by workgroups of the gate pass, in its LDS, and one more; three heads: the gate pass'
    # workgroups start at an id that is no multiple of eight
    w = with_shape(WORKLOADS["cfg1"], name=f"lists-L{L}", B=1, H=3, L=L, d=64, block=8, topk=5, window=11, len_lo=L - 50, len_hi=L,
                   seed=78)
    run_case(w, backward=True, gate_scale=0.4)


@pytest.mark.parametrize("L", [8192, 8193, 8392])
def test_gate_sums_beside_the_backward_of_long_histories(L):
    # bf16, d = 64, block 32: 64 partial sums to a head and row, as many as are taken at a time, and more; the second row's first
    # ones are of padding
    w = with_shape(WORKLOADS["cfg3"], name=f"gate-L{L}", B=2, H=2, L=L, topk=3, window=40, len_lo=300, len_hi=L, seed=79)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:] = [L, 300]
    run_case(w, x=x, backward=True, gate_scale=0.4)


def test_edge_cases():
    base = with_shape(WORKLOADS["cfg1"], name="edge", B=5, H=2, L=50, seed=301)
    x = make_inputs(base, want_dO=True)
    x.valid_len[:] = [0, 1, 50, 8, 9]          # empty row, single item, full row, one block, block + 1
    run_case(base, x=x, backward=True, check_dense=True)
    # top-k covering all blocks and window >= L: both branches are dense causal attention
    w = with_shape(base, name="dense-limit", topk=base.NB, window=base.L)
    x2, sel, f, _ = run_case(w, x=make_inputs(w, want_dO=True), backward=True, check_dense=True)
    dv = Dev(x2)
    Od, _ = B.dense_causal_fwd(params(w), dv.Q, dv.K, dv.V, dv.vl)
    torch.cuda.synchronize()
    assert_close(host(f.o_lt), host(Od), 1e-5, "o_lt vs dense kernel")
    assert_close(host(f.o_st), host(Od), 1e-5, "o_st vs dense kernel")
    # every row empty: all outputs and gradients are zero, nothing faults (each kernel family)
    for wz in (with_shape(base, name="all-empty", B=2), with_shape(base, name="all-empty-scalar", B=2, d=64),
               with_shape(WORKLOADS["cfg3"], name="all-empty-mc", B=2, H=2, L=32 * 5 + 7)):
        xz = make_inputs(wz, want_dO=True)
        xz.valid_len[:] = 0
        _, selz, fz, gz = run_case(wz, x=xz, backward=True, check_dense=True)
        assert int((selz != -1).sum()) == 0
        for t in (fz.O, fz.o_lt, fz.o_st, gz.dQ, gz.dK, gz.dV, gz.d_gate_w, gz.d_gate_b):
            assert float(t.float().abs().max()) == 0.0
    # k = 1 (own block only), w = 1 (self only), k larger than the number of blocks
    run_case(with_shape(base, name="k1w1", topk=1, window=1), backward=True)
    run_case(with_shape(base, name="kbig", topk=12, window=200), backward=True)
    # the "unbounded window" idiom: the largest int, in each kernel family
    run_case(with_shape(base, name="wmax", topk=2, window=2**31 - 1), backward=True)
    run_case(with_shape(base, name="wmax-scalar", topk=2, window=2**31 - 1, d=64), backward=True)
    run_case(with_shape(WORKLOADS["cfg3"], name="wmax-mc", B=2, H=2, L=32 * 6 + 5, len_lo=60, len_hi=32 * 6 + 5, topk=2,
                        window=2**31 - 1), backward=True)


@pytest.mark.parametrize("dtype,d,H,L,b,k,w,sblk", [
    ("fp32", 8, 8, 100, 16, 4, 8, 1),     # the paper's own setting: hidden 64 over 8 heads, length 100 (App. E)
    ("fp32", 16, 8, 200, 16, 4, 8, 1),    # ML-1M: hidden 128 over 8 heads, length 200
    ("bf16", 8, 8, 200, 16, 4, 8, 0),
    ("bf16", 16, 4, 333, 32, 3, 40, 0),
    ("fp32", 8, 2, 77, 8, 2, 5, 4),
    ("fp32", 16, 2, 500, 64, 5, 70, 0),
])
def test_small_head_dims(dtype, d, H, L, b, k, w, sblk):
    wl = with_shape(WORKLOADS["cfg1"], name=f"d{d}-{dtype}", B=6, H=H, L=L, d=d, block=b, topk=k, window=w, dtype=dtype,
                    len_lo=0, len_hi=L, qkv_scaled=(dtype == "bf16"), seed=1700 + d + L, stis_block=sblk)
    run_case(wl, backward=True, check_dense=True, gate_scale=0.4)


@pytest.mark.parametrize("dtype,d,b,L,k", [
    ("fp32", 32, 8, 203, 3),
    ("fp32", 8, 16, 200, 4),
    ("bf16", 64, 64, 1000, 5),
    ("bf16", 16, 32, 417, 2),
    ("fp32", 16, 8, 517, 5),     # 65 blocks: a thread per candidate, for the last block alone
    ("bf16", 64, 32, 4101, 6),   # 129: for every block
])
def test_select_with_compressed_keys(dtype, d, b, L, k):
    # blossom_select_blocks_cmp: the caller's compressed keys replace the block means (Eq. 9 with a
    # learnable phi); bit-exact against the oracle, in both the full and the serving mode
    w = with_shape(WORKLOADS["cfg1"], name=f"cmp-{dtype}-{d}", B=5, H=3, L=L, d=d, block=b, topk=k, dtype=dtype,
                   len_lo=1, len_hi=L, qkv_scaled=(dtype == "bf16"), seed=4100 + d + b)
    x = make_inputs(w)
    rng = np.random.default_rng(w.seed + 1)
    Kc = rng.standard_normal((w.B, w.H, w.NB, d)).astype(np.float32)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Kc_dev = torch.from_numpy(Kc).cuda().to(tdt)
    Kc = Kc_dev.float().cpu().numpy()   # what the kernel sees, exactly
    dv = Dev(x)
    sel = B.select_blocks_cmp(params(w), dv.Q, Kc_dev, dv.vl)
    ref = oracle.select_blocks_cmp(x.Q, Kc, x.valid_len, b, k)
    np.testing.assert_array_equal(sel.cpu().numpy(), ref)
    # serving mode: only the last query block's row is written, and it is the same row
    sel_last = torch.full_like(sel, -7)
    B.select_blocks_cmp(params(w, last_block_only=1), dv.Q, Kc_dev, dv.vl, sel=sel_last)
    assert torch.equal(sel_last[:, :, -1], sel[:, :, -1]) and bool((sel_last[:, :, :-1] == -7).all())


@pytest.mark.parametrize("name,shape,scale", [
    ("cfg1", dict(), 0.4),                                                   # fp32 matrix instructions
    ("cfg1", dict(d=64), 0.4),                                               # scalar kernels, fp32
    ("cfg3", dict(B=3, L=32 * 7 + 5, len_lo=30, len_hi=32 * 7 + 5), 0.07),   # matrix cores, b = 32
    ("cfg4", dict(B=2, H=2, L=64 * 5 + 9, len_lo=90, len_hi=64 * 5 + 9), 0.25),  # matrix cores, b = 64, sharper than 1/sqrt(d)
])
def test_caller_softmax_scale(name, shape, scale):
    # softmax_scale > 0 replaces the default 1/sqrt(d) in every kernel family, forward and backward
    run_case(with_shape(WORKLOADS[name], name=name + "-scale", **shape), backward=True, check_dense=True,
             gate_scale=0.4, scale=scale)


def test_forced_gate():
    w = WORKLOADS["cfg1"]
    x = make_inputs(w, want_dO=True)
    dv = Dev(x)
    p = params(w, save_for_bwd=1)
    sel = B.select_blocks(p, dv.Q, dv.K, dv.vl)
    zero = torch.zeros_like(dv.gw)
    big = torch.full_like(dv.gb, 1e4)
    f1 = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, zero, big)
    f0 = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, zero, -big)
    fn = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, zero, None)
    torch.cuda.synchronize()
    assert torch.equal(f1.O, f1.o_lt) and torch.equal(f0.O, f0.o_st)
    assert_close(host(fn.O), 0.5 * (host(fn.o_lt) + host(fn.o_st)), 1e-6, "gate_b = NULL")
    # backward: a NULL bias is a zero bias, and a NULL d_gate_b is simply not written
    fz = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, torch.zeros_like(dv.gb))
    fN = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, None)
    gz = B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, torch.zeros_like(dv.gb), fz, dv.dO)
    outN = B.BwdOut(torch.empty_like(gz.dQ), torch.empty_like(gz.dK), torch.empty_like(gz.dV),
                    torch.empty_like(gz.d_gate_w), None)
    gN = B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, None, fN, dv.dO, out=outN)
    torch.cuda.synchronize()
    assert torch.equal(fz.O, fN.O)
    for a, b_ in ((gz.dQ, gN.dQ), (gz.dK, gN.dK), (gz.dV, gN.dV), (gz.d_gate_w, gN.d_gate_w)):
        assert torch.equal(a, b_)


def test_selection_only_large_and_invariances():
    # selection at every full size is cheap for the oracle: compare all of it
    for name in ("cfg3", "cfg4"):
        w = WORKLOADS[name]
        x = make_inputs(w, want_dO=False)
        dv = Dev(x)
        sel = B.select_blocks(params(w), dv.Q, dv.K, dv.vl)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(sel.cpu().numpy(),
                                      oracle.select_blocks(x.Q, x.K, x.valid_len, w.block, w.topk))
        del dv
        torch.cuda.empty_cache()
    # planted ties: identical key blocks must resolve to the lowest index
    w = with_shape(WORKLOADS["cfg1"], name="ties", B=2, H=2, L=64, d=32, block=8, topk=3, len_lo=64, len_hi=64,
                   seed=401)
    x = make_inputs(w)
    x.K[:, :, 16:24] = x.K[:, :, 0:8]
    x.K[:, :, 40:48] = x.K[:, :, 0:8]
    dv = Dev(x)
    sel = B.select_blocks(params(w), dv.Q, dv.K, dv.vl)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(sel.cpu().numpy(), oracle.select_blocks(x.Q, x.K, x.valid_len, 8, 3))


def test_backward_passes_one_at_a_time_equal_the_full_call():
    for w in (WORKLOADS["cfg1"], with_shape(WORKLOADS["cfg3"], B=3)):
        x = make_inputs(w, want_dO=True)
        dv = Dev(x)
        p = params(w, save_for_bwd=1)
        sel = B.select_blocks(p, dv.Q, dv.K, dv.vl)
        f = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb)
        full = B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO)
        ws = torch.empty(B.workspace_bytes(p, B.WS_BWD), dtype=torch.uint8, device="cuda")
        parts = None
        for st in (B.BWD_GATE, B.BWD_INVERSE, B.BWD_DQ, B.BWD_DKV):
            parts = B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO, out=parts, ws=ws, stages=st)
        torch.cuda.synchronize()
        for a, b_ in ((full.dQ, parts.dQ), (full.dK, parts.dK), (full.dV, parts.dV),
                      (full.d_gate_w, parts.d_gate_w), (full.d_gate_b, parts.d_gate_b)):
            assert torch.equal(a, b_)


def test_step_under_a_hip_graph():
    # The library allocates nothing, clears nothing with memset nodes and never synchronises, so a whole
    # training step can be captured once and replayed: every replay (with new inputs copied into the
    # captured buffers, and eager work between the replays) must reproduce the eager results bit for bit.
    for w in (WORKLOADS["cfg1"], with_shape(WORKLOADS["cfg3"], B=2, H=2, L=32 * 7 + 9, len_lo=50, len_hi=32 * 7 + 9)):
        p = params(w, save_for_bwd=1)
        xs = [make_inputs(with_shape(w, seed=w.seed + 31 * i), want_dO=True) for i in range(3)]
        dv = Dev(xs[0])
        ws_sel = torch.empty(max(1, B.workspace_bytes(p, B.WS_SELECT)), dtype=torch.uint8, device="cuda")
        ws_bwd = torch.empty(max(1, B.workspace_bytes(p, B.WS_BWD)), dtype=torch.uint8, device="cuda")
        sel = B.select_blocks(p, dv.Q, dv.K, dv.vl, ws=ws_sel)
        f = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb)
        g = B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO, ws=ws_bwd)
        torch.cuda.synchronize()

        def step():
            B.select_blocks(p, dv.Q, dv.K, dv.vl, sel=sel, ws=ws_sel)
            B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, out=f)
            B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO, out=g, ws=ws_bwd)

        graph = torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            step()  # warm-up on the capture stream
            side.synchronize()
            with torch.cuda.graph(graph, stream=side):
                step()
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        for x in xs[::-1] + xs:
            fresh = Dev(x)
            for dst, src in ((dv.Q, fresh.Q), (dv.K, fresh.K), (dv.V, fresh.V), (dv.dO, fresh.dO), (dv.vl, fresh.vl)):
                dst.copy_(src)
            step()  # eager
            torch.cuda.synchronize()
            want = [t.clone() for t in (sel, f.O, f.o_lt, f.o_st, f.lse_lt, f.lse_st, g.dQ, g.dK, g.dV, g.d_gate_w, g.d_gate_b)]
            for t in (sel, f.O, f.o_lt, f.o_st, f.lse_lt, f.lse_st, g.dQ, g.dK, g.dV, g.d_gate_w, g.d_gate_b):
                t.fill_(1)  # eager work between the replays, and proof that the replay rewrites everything
            graph.replay()
            torch.cuda.synchronize()
            for a, b_ in zip(want, (sel, f.O, f.o_lt, f.o_st, f.lse_lt, f.lse_st, g.dQ, g.dK, g.dV, g.d_gate_w, g.d_gate_b)):
                assert torch.equal(a, b_)
