"""Timed cases of the Blossom attention path, each a call sequence that a user's program makes per batch.

A case names a kind of call, a shape and the options; the shapes are those of the repository's five workloads
(`inputs.WORKLOADS`), of `bench.py --stage positions` and of the efficiency-study shapes of the documentation, plus
generic odd sizes.  Inputs, output buffers and workspaces live on the GPU and are made once per state, as the C ABI asks
of its callers (the library owns no memory); a pass is the calls themselves.

kinds:
  infer      select_blocks, attn_fwd                                      scoring a batch
  serve      the same with last_block_only: only the last position's representation is scored
  train      select_blocks, attn_fwd (saving), attn_bwd                   one attention layer of a training step
  layer      rope_select_blocks, attn_fwd (saving), out_proj_ln, attn_bwd with the rotation undone
  positions  select_positions, attn_fwd_positions, attn_bwd_positions     the selection rule per query position
"""
import math

import torch

from paper_2512_13368_amd import binding as B
from paper_2512_13368_amd.inputs import rope_tables


def _case(name, kind, batch, heads, length, dim, block, topk, window, dtype, len_lo=0, stis=0, stis_block=0, groups=0):
    """len_lo: shortest history of a batch row (0: every row is full); stis: the short-term mask (0 local window, 1 all of
    Eq. 15, 2 the bidirectional form); stis_block: its mask block; groups: key/value heads of the per-position kind."""
    c = {"kind": kind, "B": batch, "H": heads, "L": length, "d": dim, "block": block, "topk": topk, "window": window,
         "dtype": dtype, "len_lo": len_lo or length, "stis": stis, "stis_block": stis_block, "groups": groups}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a handful of short histories: nothing but launches and the host path (workload cfg1)
        _case("tiny_infer_fp32", "infer", 4, 2, 50, 32, 8, 2, 8, "fp32", len_lo=10),
        # a training batch of short histories, hidden size 64 over two heads (workload cfg2)
        _case("short_train_fp32", "train", 256, 2, 200, 32, 16, 4, 16, "fp32", len_lo=20),
        # the same batch in bf16 for a backbone without a causal mask
        _case("short_train_bidir_bf16", "train", 256, 2, 200, 32, 16, 4, 16, "bf16", len_lo=20, stis=2, stis_block=16),
        # the paper's own training batch: 2048 rows, hidden size 128 over 8 heads, mask block 1
        _case("paper_train_fp32", "train", 2048, 8, 200, 16, 16, 4, 8, "fp32", len_lo=20, stis=1, stis_block=1),
        # the selection rule as printed, hidden size 64 over 8 heads sharing 4 key/value heads
        _case("positions_train_fp32", "positions", 2048, 8, 200, 8, 16, 4, 8, "fp32", len_lo=20, stis=1, stis_block=1,
              groups=4),
        # the efficiency study: 32 full histories of 2000 items at the paper's hyperparameters
        _case("study_train_fp32", "train", 32, 8, 2000, 8, 16, 4, 8, "fp32", stis=1, stis_block=1),
        # scoring and training at a history of 1024 with ragged rows (workloads cfg3, cfg5)
        _case("mid_infer_bf16", "infer", 128, 4, 1024, 64, 32, 8, 64, "bf16", len_lo=100),
        _case("mid_train_bf16", "train", 128, 4, 1024, 64, 32, 8, 64, "bf16", len_lo=100),
        # a whole layer at an odd length: rotary embedding, all of Eq. 15, projection, residual and LayerNorm
        _case("layer_train_bf16", "layer", 32, 8, 1997, 64, 32, 8, 64, "bf16", len_lo=200, stis=1, stis_block=32),
        # online serving of long histories: the last position only
        _case("serve_bf16", "serve", 16, 8, 8192, 64, 64, 16, 128, "bf16"),
        # long histories, scored and trained (workload cfg4)
        _case("long_infer_bf16", "infer", 16, 8, 8192, 64, 64, 16, 128, "bf16"),
        _case("long_train_bf16", "train", 16, 8, 8192, 64, 64, 16, 128, "bf16"),
    ]


def _log(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    regime = rng.choice(["short", "short", "positions", "study", "mid", "mid", "layer", "serve", "long"])
    if regime in ("short", "positions"):
        length, dim, heads = rng.randint(50, 200), rng.choice([8, 16, 32]), rng.choice([2, 4, 8])
        batch = _log(rng, 4, min(2048, 24_000_000 // (length * dim * heads)))
        len_lo, dtype = max(1, length // 10), rng.choice(["fp32", "fp32", "bf16"])
        block, topk, window = rng.choice([8, 16]), rng.randint(2, 4), rng.randint(8, 16)
        if regime == "positions":
            return _case(None, "positions", batch, heads, length, dim, 16, topk, window, dtype, len_lo, 1, 1, heads // 2)
        stis = rng.choice([0, 1, 2])
        return _case(None, rng.choice(["infer", "train"]), batch, heads, length, dim, block, topk, window, dtype, len_lo,
                     stis, 0 if stis == 0 else 1 if stis == 1 else block)
    if regime == "study":
        return _case(None, rng.choice(["infer", "train"]), rng.randint(8, 32), 8, rng.randint(500, 2000),
                     rng.choice([8, 16]), 16, 4, 8, "fp32", 0, 1, 1)
    if regime == "serve":
        return _case(None, "serve", _log(rng, 1, 16), rng.choice([4, 8]), _log(rng, 500, 8192), 64, rng.choice([32, 64]),
                     rng.randint(8, 16), rng.choice([64, 128]), "bf16")
    if regime == "long":
        length, heads = rng.randint(2048, 8192), rng.choice([4, 8])
        batch = _log(rng, 1, min(16, 1_000_000 // (length * heads)))
        return _case(None, rng.choice(["infer", "train"]), batch, heads, length, 64, 64, rng.randint(8, 16),
                     rng.choice([64, 128]), "bf16")
    length, heads = _log(rng, 200, 2000), rng.choice([4, 8])
    batch = _log(rng, 8, min(128, 500_000 // (length * heads)))
    if regime == "layer":
        stis = rng.choice([0, 1])
        return _case(None, "layer", batch, heads, length, 64, 32, rng.randint(4, 8), 64, "bf16", length // 10, stis,
                     32 * stis)
    return _case(None, rng.choice(["infer", "train"]), batch, heads, length, 64, 32, rng.randint(4, 8),
                 rng.choice([32, 64]), "bf16", length // 10)


# compression blocks of the per-position rule: 32 positions every 16
_CMP_BLOCK, _CMP_STRIDE = 32, 16


class _State:
    pass


def prepare(case, seed):
    s, dev = _State(), torch.device("cuda:0")
    n, H, L, d = case["B"], case["H"], case["L"], case["d"]
    bf16 = case["dtype"] == "bf16"
    dt = torch.bfloat16 if bf16 else torch.float32
    g = torch.Generator(device=dev).manual_seed(seed)
    kind = s.kind = case["kind"]
    train = kind in ("train", "layer", "positions")
    G = s.G = case["groups"] or H
    # projections of normalised activations: unit variance, or scaled by 1/sqrt(d) as in the bf16 workloads
    qkv = 1.0 / math.sqrt(d) if bf16 and d == 64 else 1.0

    def normal(*shape, scale=1.0, dtype=dt):
        return torch.randn(shape, generator=g, device=dev, dtype=torch.float32).mul_(scale).to(dtype)

    def new(*shape, dtype=dt):
        return torch.empty(shape, dtype=dtype, device=dev)

    def bytes_(count):
        return torch.empty(max(16, count), dtype=torch.uint8, device=dev)

    s.Q = normal(n, H, L, d, scale=qkv)
    s.K, s.V = normal(n, G, L, d, scale=qkv), normal(n, G, L, d, scale=qkv)
    s.dO = normal(n, H, L, d) if train else None
    s.valid_len = torch.randint(case["len_lo"], L + 1, (n,), generator=g, device=dev, dtype=torch.int32)
    s.gate_w, s.gate_b = normal(H, 2 * d, scale=0.02, dtype=torch.float32), normal(H, scale=0.02, dtype=torch.float32)
    p = s.p = B.Params(n, H, L, d, case["block"], case["topk"], case["window"], B.BF16 if bf16 else B.F32,
                       stis_mode=case["stis"], stis_block=case["stis_block"],
                       save_for_bwd=int(train and kind != "positions"), last_block_only=int(kind == "serve"))

    s.fwd = B.FwdOut(new(n, H, L, d))
    if train:
        s.fwd.o_lt, s.fwd.o_st = new(n, H, L, d, dtype=torch.float32), new(n, H, L, d, dtype=torch.float32)
        s.fwd.lse_lt, s.fwd.lse_st = new(n, H, L, dtype=torch.float32), new(n, H, L, dtype=torch.float32)
        s.bwd = B.BwdOut(new(n, H, L, d), new(n, G, L, d), new(n, G, L, d), new(H, 2 * d, dtype=torch.float32),
                         new(H, dtype=torch.float32))
        s.ws_bwd = bytes_(B.workspace_bytes(p, B.WS_BWD))
    if kind == "positions":
        s.sel = new(n, G, L, p.topk, dtype=torch.int32)
        s.ws_sel = bytes_(B.select_positions_workspace_bytes(p, G, _CMP_BLOCK, _CMP_STRIDE))
    else:
        s.sel = new(n, H, p.NB, p.topk, dtype=torch.int32)
        s.ws_sel = bytes_(B.workspace_bytes(p, B.WS_SELECT))
    if kind == "layer":
        width = s.width = H * d
        s.rope = tuple(torch.from_numpy(t).to(dev) for t in rope_tables(L, d))
        s.Q_rot, s.K_rot = new(n, H, L, d), new(n, H, L, d)
        s.W_O_t, s.bias = normal(width, width, scale=width ** -0.5), normal(width, scale=0.02, dtype=torch.float32)
        s.H_prev, s.S = normal(n, L, width), new(n, L, width)
        s.gamma = 1.0 + normal(width, scale=0.02, dtype=torch.float32)
        s.beta = normal(width, scale=0.02, dtype=torch.float32)
    return s


def run(s):
    p, f = s.p, s.fwd
    if s.kind == "positions":
        B.select_positions(p, s.G, _CMP_BLOCK, _CMP_STRIDE, s.Q, s.K, s.valid_len, sel_pos=s.sel, ws=s.ws_sel)
        B.attn_fwd_positions(p, s.G, s.Q, s.K, s.V, s.valid_len, s.sel, s.gate_w, s.gate_b, out=f)
        g = B.attn_bwd_positions(p, s.G, s.Q, s.K, s.V, s.valid_len, s.sel, s.gate_w, s.gate_b, f, s.dO, out=s.bwd,
                                 ws=s.ws_bwd)
        return _trained(s, f, g)
    if s.kind == "layer":
        B.rope_select_blocks(p, s.Q, s.K, *s.rope, s.valid_len, Q_rot=s.Q_rot, K_rot=s.K_rot, sel=s.sel, ws=s.ws_sel)
        B.attn_fwd(p, s.Q_rot, s.K_rot, s.V, s.valid_len, s.sel, s.gate_w, s.gate_b, out=f)
        S, mean, rstd = B.out_proj_ln(p, s.width, f.O, s.W_O_t, s.H_prev, s.gamma, s.beta, 1e-5, bias=s.bias, S=s.S,
                                      want_stats=True)
        g = B.attn_bwd(p, s.Q_rot, s.K_rot, s.V, s.valid_len, s.sel, s.gate_w, s.gate_b, f, s.dO, out=s.bwd, ws=s.ws_bwd,
                       rope=s.rope)
        return dict(_trained(s, f, g), Q_rot=s.Q_rot, K_rot=s.K_rot, S=S, mean=mean, rstd=rstd)
    B.select_blocks(p, s.Q, s.K, s.valid_len, sel=s.sel, ws=s.ws_sel)
    B.attn_fwd(p, s.Q, s.K, s.V, s.valid_len, s.sel, s.gate_w, s.gate_b, out=f)
    if s.kind == "serve":  # what the call writes: the last query block
        lo = (p.NB - 1) * p.block
        return {"sel": s.sel[:, :, p.NB - 1], "O": f.O[:, :, lo:]}
    if s.kind == "infer":
        return {"sel": s.sel, "O": f.O}
    g = B.attn_bwd(p, s.Q, s.K, s.V, s.valid_len, s.sel, s.gate_w, s.gate_b, f, s.dO, out=s.bwd, ws=s.ws_bwd)
    return _trained(s, f, g)


def _trained(s, f, g):
    return {"sel": s.sel, "O": f.O, "o_lt": f.o_lt, "o_st": f.o_st, "lse_lt": f.lse_lt, "lse_st": f.lse_st,
            "dQ": g.dQ, "dK": g.dK, "dV": g.dV, "d_gate_w": g.d_gate_w, "d_gate_b": g.d_gate_b}


def _pairs(case, length):
    """Unmasked (query, key) pairs of both branches in one (row, head) of `length` valid positions, the last block alone
    in the serving kind.  Block boundaries are counted from the first valid position: an average over its offset."""
    b, k, w, L, stis = case["block"], case["topk"], case["window"], case["L"], case["stis"]
    blk = case["stis_block"]
    first = max(0, length - b) if case["kind"] == "serve" else 0
    total = 0
    for i in range(first, length):
        blocks, own = i // b, i % b + 1
        if stis == 2:
            total += min(k, -(-length // b)) * b
            near = min(w - 1, i) + 1 + min(w - 1, length - 1 - i)
        else:
            total += min(k - 1, blocks) * b + own
            near = min(w, i + 1)
        if stis:  # whole mask blocks at power-of-two distances, as far as the window has not taken them
            reach = [2 ** e for e in range(L.bit_length()) if 2 ** e * blk >= w]
            near += sum(blk for r in reach if r * blk <= i)
            if stis == 2:
                near += sum(blk for r in reach if i + r * blk < length)
        total += near
    return total


def work(case):
    n, H, L, d, k = case["B"], case["H"], case["L"], case["d"], case["topk"]
    G = case["groups"] or H
    size = 2 if case["dtype"] == "bf16" else 4
    kind = case["kind"]
    mean_len = (case["len_lo"] + L) / 2.0
    some = sorted({case["len_lo"] + round((L - case["len_lo"]) * (q + 0.5) / 4) for q in range(4)})
    pairs = n * H * sum(_pairs(case, m) for m in some) / len(some)
    # valid positions are read once; outputs are written at every position (padding rows get zeros)
    q_in, kv_in, q_out, kv_out = n * H * mean_len * d, n * G * mean_len * d, n * H * L * d, n * G * L * d
    if kind == "serve":
        last = n * H * case["block"] * d
        keys = min(L, k * case["block"] + case["window"])  # values of the attended blocks; keys once for the selection
        moved = (q_in / mean_len * case["block"] + kv_in + n * G * keys * d + last) * size + n * H * k * 4
        return {"bytes": moved, "flops": 4.0 * d * pairs}
    rows = n * G * L if kind == "positions" else n * H * -(-L // case["block"])
    moved = (q_in + 2 * kv_in + q_out) * size + rows * k * 4
    flops = 4.0 * d * pairs
    if kind != "infer":
        saved = 2 * q_out * 4 + 2 * n * H * L * 4
        moved += saved + (q_in + q_out + 2 * kv_out) * size  # branch outputs and lse written; dO read; dQ, dK, dV written
        flops += 10.0 * d * pairs
    if kind == "layer":
        moved += (2 * n * H * L * d + 2 * n * L * H * d + (H * d) ** 2) * size + 2 * n * L * 4
        flops += 2.0 * n * L * (H * d) ** 2
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    # selected blocks are whole numbers with one right answer.  bf16: results and matrix operands carry 8 bits, each result
    # within 2e-2 of (its value + the rms); fp32: products and sums in fp32, 1e-4 by the same measure
    return {"rel": 1e-2, "max": 6e-2} if case["dtype"] == "bf16" else {"rel": 2e-5, "max": 2e-4}
