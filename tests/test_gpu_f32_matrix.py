"""GPU parity of the fp32 matrix-instruction kernels for small heads (fp32 or bf16 storage, d in {8, 16, 32}, block 8 or
16, up to 16384 positions): forward, dQ and dK/dV against the CPU oracle, with a whole head in LDS, with its tiles streamed,
at the lengths where one takes over from the other, and where the scalar-ALU kernels take over from both."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import TOL, Dev, assert_close, host, params
from paper_2512_13368_amd import binding as B
from paper_2512_13368_amd.inputs import WORKLOADS, make_inputs, rope_tables, with_shape
from test_gpu_parity import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,L,topk,window", [
    (16, 200, 4, 16),    # the short-sequence recommender shape (cfg2), with backward
    (16, 197, 4, 16),    # ragged last block
    (16, 208, 5, 40),    # 13 whole tiles
    (8, 200, 4, 8),      # block 8: two blocks per 16-row tile, the last tile half empty
    (8, 51, 2, 8),       # ragged, block 8
    (16, 16, 1, 1),      # one block, own block only, self only
    (16, 33, 3, 500),    # window beyond the sequence, top-k = number of blocks
])
def test_short_sequences_forward_backward(b, L, topk, window):
    w = with_shape(WORKLOADS["cfg2"], name=f"f32mc-b{b}-L{L}", B=7, H=3, L=L, block=b, topk=topk, window=window,
                   len_lo=1, len_hi=L, seed=900 + b + L)
    x = make_inputs(w, want_dO=True)
    # a full row, a row starting inside a block, one shorter than a block, a single item, an empty row
    x.valid_len[:5] = [L, max(1, L - b - 3), min(L, b // 2 + 1), 1, 0]
    run_case(w, x=x, backward=True, check_dense=True, gate_scale=0.4)


@pytest.mark.parametrize("Bn,H", [(130, 2), (64, 8), (171, 3), (512, 2), (513, 2)])
def test_heads_taken_by_length(Bn, H):
    # more heads than CUs: one turn and a bit, two whole turns, two and a bit, as many rows as are ordered, one more (L: from where
    # the order is used at all of them)
    w = with_shape(WORKLOADS["cfg2"], name=f"f32mc-order-B{Bn}-H{H}", B=Bn, H=H, L=210, d=8, block=16, topk=2, window=4, len_lo=1,
                   len_hi=210, seed=960 + Bn)
    x = make_inputs(w, want_dO=True)
    x.valid_len[1::3] = x.valid_len[1]                                  # lengths that many rows share
    x.valid_len[[0, 2, 5, Bn - 1]] = [210, 0, 211, -3]                  # longest, empty, past either end
    run_case(w, x=x, backward=True, gate_scale=0.4)


@pytest.mark.parametrize("d,Bn,H", [(16, 130, 2), (32, 64, 8), (8, 130, 4)])
def test_heads_taken_by_length_in_bf16(d, Bn, H):
    w = with_shape(WORKLOADS["cfg2"], name=f"f32mc-order-bf16-d{d}-B{Bn}-H{H}", B=Bn, H=H, L=150, d=d, block=16, topk=2, window=4,
                   dtype="bf16", qkv_scaled=True, len_lo=1, len_hi=150, seed=970 + d)
    x = make_inputs(w, want_dO=True)
    x.valid_len[1::3] = x.valid_len[1]
    x.valid_len[[0, 2, 5, Bn - 1]] = [150, 0, 151, -3]
    run_case(w, x=x, backward=True, gate_scale=0.4)


def test_sharp_softmax_and_holes():
    # logits large enough that a few keys take a row's whole weight; caller-built selection rows with holes are skipped
    # where they stand
    w = with_shape(WORKLOADS["cfg2"], name="f32mc-sharp", B=4, H=2, L=150, topk=5, window=24, len_lo=40, len_hi=150,
                   seed=951)
    x = make_inputs(w, want_dO=True)
    x.Q *= np.float32(3.0)

    def punch(sel):
        NB = sel.shape[2]
        for I in range(NB):
            row = sel[:, :, I]
            full = (row >= 0).sum(-1) >= 3
            row[full, 0] = NB + 2          # an id past the last block, up front
            row[full, 1] = -1              # a hole
        return sel

    run_case(w, x=x, backward=True, sel_edit=punch)


def test_rope_backward_and_serving_mode():
    w = with_shape(WORKLOADS["cfg2"], name="f32mc-rope", B=5, H=2, L=120, len_lo=10, len_hi=120, seed=977)
    x = make_inputs(w, want_dO=True)
    cos, sin = rope_tables(w.L, w.d)
    dv = Dev(x)
    cos_d, sin_d = torch.from_numpy(cos).cuda(), torch.from_numpy(sin).cuda()
    p = params(w, save_for_bwd=1)
    Q_rot, K_rot, sel = B.rope_select_blocks(p, dv.Q, dv.K, cos_d, sin_d, dv.vl)
    f = B.attn_fwd(p, Q_rot, K_rot, dv.V, dv.vl, sel, dv.gw, dv.gb)
    g = B.attn_bwd(p, Q_rot, K_rot, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO, rope=(cos_d, sin_d))
    torch.cuda.synchronize()
    Qr, Kr = oracle.rope(x.Q, cos, sin), oracle.rope(x.K, cos, sin)
    sel_ref = oracle.select_blocks(Qr, Kr, x.valid_len, w.block, w.topk)
    np.testing.assert_array_equal(sel.cpu().numpy(), sel_ref)
    flat = lambda t: host(t).reshape(w.B * w.H, *t.shape[2:])
    tol = TOL[w.dtype]
    fr = oracle.attn_fwd(Qr, Kr, x.V, x.valid_len, sel_ref, x.gate_w, x.gate_b, w.block, w.topk, w.window)
    gr = oracle.attn_bwd(Qr, Kr, x.V, x.valid_len, sel_ref, x.gate_w, x.gate_b, x.dO, w.block, w.topk, w.window)
    assert_close(flat(f.O), fr.O, tol, "O")
    assert_close(flat(g.dQ), oracle.rope_bwd(gr.dQ, cos, sin), tol, "dQ (rotated back)")
    assert_close(flat(g.dK), oracle.rope_bwd(gr.dK, cos, sin), tol, "dK (rotated back)")
    assert_close(flat(g.dV), gr.dV, tol, "dV")
    # serving mode: only the last query block is written, and it equals the full run's
    O = torch.full_like(f.O, 3.0)
    B.attn_fwd(params(w, last_block_only=1), Q_rot, K_rot, dv.V, dv.vl, sel, dv.gw, dv.gb, out=B.FwdOut(O))
    torch.cuda.synchronize()
    lo = (w.NB - 1) * w.block
    assert torch.equal(O[:, :, lo:], f.O[:, :, lo:]) and bool((O[:, :, :lo] == 3.0).all())


@pytest.mark.parametrize("d,L", [
    (32, 224),
    (32, 128), (32, 129), (32, 240), (32, 241), (32, 256), (32, 257),
    (16, 224), (16, 225), (16, 416), (16, 417), (16, 480), (16, 481),
    (8, 352), (8, 353), (8, 640), (8, 641), (8, 800), (8, 801),
    (16, 128), (16, 129), (16, 240), (16, 241), (16, 272), (16, 273),
    (8, 288), (8, 289), (8, 496), (8, 497), (8, 688), (8, 689),
])
def test_edges_of_the_resident_range(d, L):
    # the longest heads (and one position more) whose backward holds Q and dO beside K and V, whose backward holds them in
    # their place, and whose forward holds K and V; beyond, tiles are streamed
    run_case(with_shape(WORKLOADS["cfg2"], name=f"f32-d{d}-L{L}", B=3, H=2, L=L, d=d, len_lo=30, len_hi=L, seed=990),
             backward=True)


@pytest.mark.parametrize("dtype,d,b", [("fp32", 8, 16), ("bf16", 16, 8), ("bf16", 32, 16)])
def test_past_the_longest_small_head(dtype, d, b):
    # 16384 positions are the most those kernels take; here the scalar ones serve the same head sizes and blocks (d = 32, block
    # 8 in fp32: test_gpu_parity.py, test_many_blocks_backward)
    w = with_shape(WORKLOADS["cfg2"], name=f"past-{dtype}-d{d}-b{b}", B=1, H=1, L=16384 + 5, d=d, block=b, topk=3, window=b + 3,
                   dtype=dtype, qkv_scaled=(dtype == "bf16"), len_lo=16384 - 40, len_hi=16384 + 5, seed=995)
    run_case(w, backward=True, gate_scale=0.4)


@pytest.mark.parametrize("dtype,d,b,L,topk,window,sblk", [
    ("fp32", 8, 16, 197, 4, 8, 1),      # the paper's own hyperparameters: hidden 64 over 8 heads, mask block 1
    ("fp32", 16, 16, 200, 4, 8, 1),     # ML-1M head size
    ("bf16", 8, 8, 120, 3, 8, 2),       # bf16 storage, block 8, a small mask block
    ("bf16", 16, 16, 150, 4, 24, 16),   # mask block = selection block
    ("bf16", 32, 16, 200, 4, 16, 0),    # bf16 storage, plain window
    ("fp32", 32, 8, 90, 3, 8, 4),
])
def test_head_sizes_storage_types_and_full_short_term_mask(dtype, d, b, L, topk, window, sblk):
    w = with_shape(WORKLOADS["cfg2"], name=f"res-{dtype}-d{d}-b{b}-s{sblk}", B=5, H=16 // (d // 8 if d < 32 else 4),
                   L=L, d=d, block=b, topk=topk, window=window, dtype=dtype, qkv_scaled=(dtype == "bf16"), len_lo=1,
                   len_hi=L, stis_block=sblk, seed=1200 + d + b + sblk)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:4] = [L, max(1, L - b - 3), min(L, b // 2 + 1), 0]
    run_case(w, x=x, backward=True, check_dense=True, gate_scale=0.4)


def test_efficiency_study_length_1000():
    # the efficiency-study length 1000 at the paper's hyperparameters: K and V of a head would take 94 KB of LDS, its tiles
    # are streamed
    w = with_shape(WORKLOADS["cfg2"], name="res-L1000", B=8, H=8, L=1000, d=8, block=16, topk=4, window=8, len_lo=300,
                   len_hi=1000, stis_block=1, seed=1301)
    run_case(w, backward=True, pairs=[0, 7, 21, 38, 63])


def test_seeded_random_shapes_of_small_heads():
    # 60 seeded draws, up to 26 blocks (heads in LDS, and streamed at d = 32), over storage type, head size, block size, length, top-k, window, mask block and form
    rng = np.random.default_rng(4242)
    for case in range(60):
        dtype = "bf16" if rng.random() < 0.35 else "fp32"
        d = int(rng.choice([8, 16, 32]))
        b = int(rng.choice([8, 16]))
        nb = int(rng.integers(1, 27))
        L = max(2, nb * b - int(rng.integers(0, b)))
        topk = int(rng.choice([1, 2, 3, 4, 5, nb, nb + 3]))
        window = int(rng.choice([1, 2, b - 1, b, b + 1, 2 * b + 5, 3 * b, L, L + 7]))
        bidir = bool(rng.random() < 0.25)
        sblk = int(rng.choice([0, 0, b, 1, 3, 2 * b, 4, b // 2]))
        if bidir and sblk == 0:
            sblk = int(rng.choice([1, b, 4]))
        w = with_shape(WORKLOADS["cfg1"], name=f"rr{case}", B=4, H=int(rng.choice([2, 3, 16])), L=L, d=d, block=b,
                       topk=max(1, topk), window=max(1, window), dtype=dtype, len_lo=0, len_hi=L,
                       qkv_scaled=(dtype == "bf16"), seed=424200 + case, stis_block=sblk, bidir=bidir)
        x = make_inputs(w, want_dO=True)
        x.valid_len[:] = [L, int(rng.integers(0, L + 1)), int(rng.integers(0, L + 1)), min(L, 1 + int(rng.integers(0, b)))]
        same = w.topk >= w.NB and (w.window >= L or sblk >= L)
        run_case(w, x=x, backward=True, check_dense=(case % 4 == 0 and not bidir), gate_scale=0.4, branches_coincide=same)


@pytest.mark.parametrize("dtype,d,b,B_,H,L,sblk,bidir,amp", [
    ("fp32", 8, 8, 260, 8, 17, 1, False, 1),     # 2080 heads: four wavefronts and shared buffers per workgroup
    ("bf16", 32, 16, 257, 8, 31, 2, True, 1),    # the same in bf16, bidirectional, ragged in the second tile
    ("fp32", 32, 16, 3, 2, 225, 0, False, 1),    # past the resident backward at d = 32: its tiles are streamed
    ("fp32", 16, 8, 3, 2, 513, 1, False, 1),     # one item past 32 tiles: second word of a tile list
    ("fp32", 8, 16, 2, 2, 1043, 5, True, 1),     # past 64 tiles, bidirectional
    ("bf16", 16, 16, 2, 2, 1024, 16, False, 1),
    ("fp32", 16, 16, 5, 2, 150, 1, False, 30),   # logits beyond 60: the walk with row maxima, resident ...
    ("fp32", 32, 8, 2, 2, 530, 0, False, 30),    # ... and streamed
])
def test_many_heads_streamed_tiles_and_large_logits(dtype, d, b, B_, H, L, sblk, bidir, amp):
    w = with_shape(WORKLOADS["cfg2"], name=f"small-{dtype}-d{d}-b{b}-L{L}-x{amp}", B=B_, H=H, L=L, d=d, block=b,
                   topk=3, window=b + 3, dtype=dtype, qkv_scaled=(dtype == "bf16"), len_lo=1, len_hi=L,
                   stis_block=sblk, bidir=bidir, seed=1700 + d + b + L)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:2] = [L, max(1, L - b - 3)]
    x.Q *= np.float32(amp)
    pairs = None if B_ * H < 64 else [0, 1, H, B_ * H // 2 + 1, B_ * H - 1]
    run_case(with_shape(w, backward=False), x=x, pairs=pairs, backward=True, gate_scale=0.4)


@pytest.mark.parametrize("d,window,L,sblk,bidir", [
    (8, 1, 130, 1, False),     # the window is the query itself: the powers of two up to 16 come from the neighbouring tile
    (8, 2, 1100, 1, False),    # distances up to 1024, 70 tiles: two batches of four distances, two words of tiles
    (8, 5, 330, 1, True),      # d = 8, both directions: parts of the sums in the lane groups, a lane group to a distance
    (8, 3, 33, 1, False),      # ... a last tile of one row, distances past either end
    (8, 1, 2500, 1, True),     # ... streamed
    (16, 17, 300, 1, False),   # the window ends with the neighbouring tile ...
    (16, 18, 300, 1, False),   # ... one position into the next: distance 32 is then a test of the walk, 64 the first diagonal
    (16, 33, 513, 1, True),    # the table of distances is full; both directions; past 32 tiles
    (32, 31, 290, 1, False),   # streamed at d = 32
    (32, 50, 120, 1, True),    # in LDS, three tiles of window either side
    (8, 70, 400, 0, False),    # no Eq. 15: window tiles two and more away, whole and cut
    (32, 40, 1030, 2, True),   # a larger mask block: every test element by element
])
def test_window_against_powers_of_two(d, window, L, sblk, bidir):
    w = with_shape(WORKLOADS["cfg2"], name=f"pow2-d{d}-w{window}-L{L}", B=3, H=2, L=L, d=d, block=16, topk=3, window=window,
                   len_lo=1, len_hi=L, stis_block=sblk, bidir=bidir, seed=2300 + d + window + L)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:] = [L, L - 21, 40]
    run_case(with_shape(w, backward=False), x=x, backward=True, gate_scale=0.4)


@pytest.mark.parametrize("d,b,B_,H,L,sblk,bidir", [
    (32, 16, 2, 2, 416, 0, False),    # the longest bf16 heads at d = 32 whose backward is in LDS
    (32, 16, 2, 2, 500, 16, True),    # streamed
    (16, 8, 2, 2, 830, 1, False),
    (16, 16, 2, 2, 1100, 0, False),
    (32, 8, 1030, 2, 33, 1, True),    # 2060 heads: shared buffers
    (16, 16, 3, 2, 47, 3, False),
])
def test_bf16_rows_as_they_are_stored(d, b, B_, H, L, sblk, bidir):
    # products of bf16 rows on the bf16 matrix instructions, fp32 sides as three terms: the saved branch outputs and lse keep fp32's
    # accuracy against the oracle (bf16 itself would be off by 2e-3)
    w = with_shape(WORKLOADS["cfg2"], name=f"bf16-d{d}-b{b}-L{L}", B=B_, H=H, L=L, d=d, block=b, topk=3, window=b + 3, dtype="bf16",
                   qkv_scaled=True, len_lo=1, len_hi=L, stis_block=sblk, bidir=bidir, backward=False, seed=2800 + d + L)
    x = make_inputs(w, want_dO=True)
    x.valid_len[:2] = [L, max(1, L - b - 3)]
    pairs = None if B_ * H < 64 else [0, 1, H, B_ * H // 2 + 1, B_ * H - 1]
    run_case(w, x=x, pairs=pairs, backward=True, gate_scale=0.4)
    dv, p = Dev(x), params(w, save_for_bwd=1)
    f = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, B.select_blocks(p, dv.Q, dv.K, dv.vl), dv.gw, dv.gb)
    torch.cuda.synchronize()
    bh = np.asarray(pairs if pairs is not None else range(B_ * H), np.int32)
    sel = oracle.select_blocks(x.Q, x.K, x.valid_len, b, 3, bidir=bidir)
    fr = oracle.attn_fwd(x.Q, x.K, x.V, x.valid_len, sel, x.gate_w, x.gate_b, b, 3, b + 3, bh_list=bh, stis_block=sblk, bidir=bidir)
    take = lambda t: host(t).reshape(B_ * H, *t.shape[2:])[bh]
    for name in ("o_lt", "o_st", "lse_lt", "lse_st"):
        assert_close(take(getattr(f, name)), getattr(fr, name), TOL["fp32"], name)


@pytest.mark.parametrize("d,L,limit", [
    (8, 200, 2.42e-7),
    (16, 200, 2.55e-7),
    (16, 450, 2.76e-7),   # streamed
    (32, 200, 2.67e-7),
])
def test_errors_against_64_bits(d, L, limit):
    # fp32 under mask block 1, where single keys at powers of two are taken on the vector ALUs: dQ errs no more than where the matrix
    # cores formed every product (`limit`: measured so, on these inputs), and the lse little more than a result of about 5 does by
    # being rounded (2^-21 / sqrt(12) of it: 3e-8; the row's sum and its logarithm are to add no more than half as much)
    w = with_shape(WORKLOADS["cfg2"], name=f"exact-d{d}-L{L}", B=12, H=4, L=L, d=d, block=16, topk=4, window=8, len_lo=L // 10, len_hi=L,
                   stis_block=1, seed=3100 + d + L)
    x = make_inputs(w, want_dO=True)
    dv, p = Dev(x), params(w, save_for_bwd=1)
    sel = B.select_blocks(p, dv.Q, dv.K, dv.vl)
    f = B.attn_fwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb)
    g = B.attn_bwd(p, dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb, f, dv.dO)
    torch.cuda.synchronize()
    args = (x.Q, x.K, x.V, x.valid_len, sel.cpu().numpy(), x.gate_w, x.gate_b)
    fr = oracle.attn_fwd(*args, 16, 4, 8, stis_block=1)
    dQ = oracle.attn_bwd(*args, x.dO, 16, 4, 8, stis_block=1).dQ
    err = lambda got, ref: float(np.linalg.norm(host(got).reshape(ref.shape) - ref) / np.linalg.norm(ref))
    assert err(f.lse_lt, fr.lse_lt) < 4.5e-8 and err(f.lse_st, fr.lse_st) < 4.5e-8
    assert err(g.dQ, dQ) < limit


@pytest.mark.parametrize("d,L,sblk", [(32, 400, 0), (16, 400, 1), (8, 395, 0), (8, 1600, 4)])
def test_serving_mode_at_block_8(d, L, sblk):
    # two query blocks to a tile, most of their selected tiles beyond the window: a row of the last block has the same bits whether the
    # block beside it selected anything or not, and the full forward agrees with the oracle
    w = with_shape(WORKLOADS["cfg1"], name=f"serve8-d{d}-L{L}", B=6, H=3, L=L, d=d, block=8, topk=5, window=9, len_lo=40, len_hi=L,
                   stis_block=sblk, seed=3300 + d + L)
    x = make_inputs(w)
    dv = Dev(x)
    sel = B.select_blocks(params(w), dv.Q, dv.K, dv.vl)
    full = B.attn_fwd(params(w), dv.Q, dv.K, dv.V, dv.vl, sel, dv.gw, dv.gb).O
    last = torch.full_like(sel, -7)
    last[:, :, -1] = sel[:, :, -1]
    O = B.attn_fwd(params(w, last_block_only=1), dv.Q, dv.K, dv.V, dv.vl, last, dv.gw, dv.gb, out=B.FwdOut(torch.zeros_like(full))).O
    torch.cuda.synchronize()
    lo = (w.NB - 1) * 8
    assert torch.equal(O[:, :, lo:], full[:, :, lo:])
    fr = oracle.attn_fwd(x.Q, x.K, x.V, x.valid_len, sel.cpu().numpy(), x.gate_w, x.gate_b, 8, 5, 9, stis_block=sblk)
    assert_close(host(full).reshape(fr.O.shape), fr.O, TOL["fp32"], "O")


@pytest.mark.parametrize("d,b,L", [
    (16, 16, 416), (16, 16, 417), (16, 8, 416), (16, 8, 417), (16, 16, 560), (16, 16, 561), (16, 8, 560), (16, 8, 561),
    (32, 16, 224), (32, 16, 225), (32, 8, 224), (32, 8, 225), (32, 16, 416), (32, 16, 417), (32, 8, 416), (32, 8, 417),
    (32, 16, 480), (32, 16, 481), (32, 8, 480), (32, 8, 481),
])
def test_edges_of_the_resident_range_in_bf16(d, b, L):
    # rows as they are stored take half the LDS: the longest heads (and one position more) whose backward holds Q and dO beside K and V
    # (d = 32: 224; d = 16: all the backward takes), whose backward is in LDS (416) and whose forward is (560, 480)
    run_case(with_shape(WORKLOADS["cfg2"], name=f"bf16-d{d}-b{b}-L{L}", B=3, H=2, L=L, d=d, block=b, dtype="bf16", qkv_scaled=True, len_lo=30,
                        len_hi=L, seed=991), backward=True)


@pytest.mark.parametrize("dtype,d,B_,H,L", [
    ("fp32", 16, 128, 4, 129),                               # 512 heads: Q and dO beside K and V ...
    ("fp32", 16, 171, 3, 128), ("fp32", 16, 171, 3, 129),    # ... 513: up to 128, in their place beyond
    ("bf16", 16, 171, 3, 240), ("bf16", 16, 171, 3, 241),
    ("fp32", 8, 171, 3, 288), ("fp32", 8, 171, 3, 289), ("fp32", 8, 171, 3, 496), ("fp32", 8, 171, 3, 497),
])
def test_edges_of_the_resident_range_with_more_heads(dtype, d, B_, H, L):
    w = with_shape(WORKLOADS["cfg2"], name=f"{dtype}-d{d}-L{L}", B=B_, H=H, L=L, d=d, dtype=dtype, qkv_scaled=(dtype == "bf16"), len_lo=30,
                   len_hi=L, backward=False, seed=992)
    x = make_inputs(w, want_dO=True)
    run_case(w, x=x, pairs=[0, 1, B_ * H // 2 + 1, B_ * H - 1], backward=True, gate_scale=0.4)
