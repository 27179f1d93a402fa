"""What a user of this package has it do, as cases that can be timed: one rank's share of Unified
Sequence Parallel attention (ring attention of a Q shard over KV chunks), the FP8 pack and unpack of
the All-to-All payloads, and the log-sum-exp merge, all through the package's public entry points.

A case is a dict of plain values.  "op" is one of

  "attn"     usp_ring_attn_fwd.  B, H, d, Sq; n chunks of `chunk` keys, the last one of `last` keys;
             dtype of Q and O; kv = "same" or "fp8" (E4M3 codes with a scale per head and token);
             masked = dead keys at the end of the sequence (padding of a prompt); outliers = 1 % of
             the entries x20; mode = "resident" (every chunk at hand) or "prefetch" (the ring's
             transfers ride in the call); layout = "bhsd" (dense) or "bshd" (views of [B, S, H, d])
  "payload"  usp_fp8_quant of a [rows, cols] payload, then usp_fp8_dequant of what arrived
  "a2a"      the same from the sequence-sharded into the head-sharded layout of the All-to-All
             (usp_fp8_quant_mapped, usp_fp8_dequant_mapped), one scale per head and token
  "merge"    usp_lse_merge of two partial results
"""
import torch

import paper_2602_10940_amd as usp

DEV = "cuda:0"
DT = {"bf16": torch.bfloat16, "f32": torch.float32}
OUTLIER_FRAC, OUTLIER_MUL = 0.01, 20.0


def _attn(name, B, H, d, Sq, n, chunk, last=None, dtype="bf16", kv="same", masked=0, outliers=False, mode="resident",
          layout="bhsd"):
    case = {"op": "attn", "B": B, "H": H, "d": d, "Sq": Sq, "n": n, "chunk": chunk, "last": chunk if last is None else last,
            "dtype": dtype, "kv": kv, "masked": masked, "outliers": outliers, "mode": mode, "layout": layout}
    return dict(case, name=name) if name else case


def listed():
    return [
        # a model's smallest attention at fp32, on two ranks: what a first run or a unit test of a user's program calls
        _attn("tiny_f32_r2", 1, 2, 64, 128, 2, 128, dtype="f32"),
        # FLUX-1024 on Ulysses ranks alone: 4096 image + 512 text tokens in one chunk
        _attn("flux1024_u", 1, 24, 128, 4608, 1, 4608),
        # the same model on eight Ulysses ranks: three heads are left to a rank
        _attn("flux1024_u8", 1, 3, 128, 4608, 1, 4608),
        # the same model on a ring of four with FP8 K/V payloads
        _attn("flux1024_r4_fp8", 1, 24, 128, 1152, 4, 1152, kv="fp8", mode="prefetch"),
        # FLUX-2048 on Ulysses 2 x ring 8, bf16 payloads, the next chunk under way during the compute
        _attn("flux2048_u2r8", 1, 12, 128, 2112, 8, 2112, mode="prefetch"),
        # Qwen-Image-like shard on a ring of two: padded prompt, outliers, FP8 K/V
        _attn("qwen_r2", 1, 24, 128, 4096, 2, 4096, kv="fp8", masked=390, outliers=True),
        # an image and a prompt whose token count divides by nothing, Ulysses 2 x ring 2
        _attn("ragged_u2r2", 1, 12, 128, 2215, 2, 2215, 2214, mode="prefetch"),
        # head dimension 64, two batch entries (guidance), image and a 77-token prompt in [B, S, H, d] storage
        _attn("joint_d64", 2, 24, 64, 1101, 1, 1101, layout="bshd"),
        # a head dimension the matrix layouts do not divide evenly
        _attn("image_d72", 2, 16, 72, 1024, 1, 1024),
        # the All-to-All payload of one FLUX-1024 tensor, a scale per token: pack, then unpack
        {"name": "payload_flux1024", "op": "payload", "rows": 4608, "cols": 3072, "dtype": "bf16"},
        # the same exchange through the layouts of eight ranks, a scale per head and token, an odd shard
        {"name": "a2a_heads", "op": "a2a", "B": 1, "H": 24, "S": 577, "d": 128, "peers": 8, "dtype": "bf16"},
        # one ring step's merge as Algorithm 2 writes it, on the FLUX-1024 ring-of-four state
        {"name": "merge_flux1024_r4", "op": "merge", "rows": 27648, "d": 128, "dtype": "bf16"},
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


# no drawn attention is more work than the largest listed one of its kind
_MOST_FLOPS = 4.0 * 24 * 4096 * 8192 * 128
_MOST_FLOPS_GENERAL = 4.0 * 2 * 16 * 1024 * 1024 * 72


def _draw_attn(rng, fp8):
    d = 64 if rng.random() < 0.25 else 128
    while True:
        B, H = rng.choice([1, 1, 1, 2]), _log(rng, 1, 24)
        n = rng.choice([1, 1, 2, 2, 3, 4, 6, 8])
        chunk = _log(rng, 64, 4608)
        if rng.random() < 0.5:
            chunk = (chunk + 63) // 64 * 64
        # a rank holds as many queries as keys, give or take a token; cross attention may hold any number
        Sq = chunk if rng.random() < 0.7 else _log(rng, 64, 4608)
        if 4.0 * B * H * Sq * n * chunk * d <= _MOST_FLOPS and n * chunk <= 17000:
            break
    last = chunk if chunk % 64 == 0 or rng.random() < 0.3 else chunk - rng.randrange(min(n, chunk - 1))
    keys = (n - 1) * chunk + last
    masked = rng.randrange(1, max(2, keys // 8)) if rng.random() < 0.3 else 0
    mode = "prefetch" if n > 1 and rng.random() < 0.5 else "resident"
    layout = "bshd" if n == 1 and not fp8 and rng.random() < 0.4 else "bhsd"
    return _attn(None, B, H, d, Sq, n, chunk, last, kv="fp8" if fp8 else "same", masked=masked, outliers=rng.random() < 0.2,
                 mode=mode, layout=layout)


def _draw_general(rng):
    """fp32 inputs, and bf16 head dimensions other than 64 and 128."""
    dtype = rng.choice(["f32", "bf16"])
    d = rng.choice([32, 64, 96, 128]) if dtype == "f32" else rng.choice([40, 72, 80, 96, 112, 160])
    while True:
        B, H, n, Sq, chunk = rng.choice([1, 2]), _log(rng, 2, 24), rng.choice([1, 1, 2, 4]), _log(rng, 64, 2048), _log(rng, 64, 2048)
        if 4.0 * B * H * Sq * n * chunk * d <= _MOST_FLOPS_GENERAL:
            break
    return _attn(None, B, H, d, Sq, n, chunk, dtype=dtype, masked=rng.randrange(1, chunk // 2) if rng.random() < 0.3 else 0)


def draw(rng):
    kind = rng.random()
    if kind < 0.35:
        return _draw_attn(rng, fp8=False)
    if kind < 0.55:
        return _draw_attn(rng, fp8=True)
    if kind < 0.67:
        return _draw_general(rng)
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    if kind < 0.80:
        # from one head's rows to three tensors of FLUX-1024 at once; cols past 4096 are rows of a wider model
        rows, cols = _log(rng, 64, 13824), 8 * _log(rng, 8, 768)
        return {"op": "payload", "rows": rows, "cols": cols, "dtype": dtype}
    if kind < 0.90:
        peers = rng.choice([2, 4, 8])
        return {"op": "a2a", "B": rng.choice([1, 2]), "H": peers * rng.randint(1, 24 // peers), "S": _log(rng, 64, 4608) // rng.choice([1, 2]),
                "d": rng.choice([64, 128, 128]), "peers": peers, "dtype": dtype}
    return {"op": "merge", "rows": _log(rng, 256, 98304), "d": rng.choice([64, 128, 128, 72, 160]), "dtype": dtype}


# ---------------------------------------------------------------------------------------------------
def _a2a_map(case):
    """Rows as (peer, batch, head of the peer, token): strides of the two tensors in elements, of the codes in rows."""
    B, H, S, d, N = case["B"], case["H"], case["S"], case["d"], case["peers"]
    Hn = H // N
    return {"n": (N, B, Hn, S), "dense": (B * Hn * S, Hn * S, S, 1),
            "seq_sharded": (Hn * S * d, H * S * d, S * d, d), "head_sharded": (S * d, Hn * N * S * d, N * S * d, d)}


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)

    def normal(*shape, dtype=torch.float32):
        return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).to(dtype)

    dt = DT[case["dtype"]]
    if case["op"] == "payload":
        rows, cols = case["rows"], case["cols"]
        return {"case": case, "x": normal(rows, cols, dtype=dt), "q": torch.empty((rows, cols), dtype=torch.uint8, device=DEV),
                "s": torch.empty((rows,), device=DEV), "y": torch.empty((rows, cols), dtype=dt, device=DEV)}
    if case["op"] == "a2a":
        B, H, S, d, N = case["B"], case["H"], case["S"], case["d"], case["peers"]
        rows = B * H * S
        return {"case": case, "x": normal(B, H, S, d, dtype=dt), "map": _a2a_map(case),
                "q": torch.empty((rows, d), dtype=torch.uint8, device=DEV), "s": torch.empty((rows,), device=DEV),
                "y": torch.empty((B, H // N, N * S, d), dtype=dt, device=DEV)}
    if case["op"] == "merge":
        rows, d = case["rows"], case["d"]
        return {"case": case, "o1": normal(rows, d, dtype=dt), "o2": normal(rows, d, dtype=dt), "l1": normal(rows), "l2": normal(rows),
                "o": torch.empty((rows, d), dtype=dt, device=DEV), "l": torch.empty((rows,), device=DEV)}

    B, H, d, Sq = case["B"], case["H"], case["d"], case["Sq"]
    lens = [case["chunk"]] * (case["n"] - 1) + [case["last"]]

    def tensor(tokens):
        x = normal(B, tokens, H, d) if case["layout"] == "bshd" else normal(B, H, tokens, d)
        if case["outliers"]:
            x = torch.where(torch.rand(x.shape, generator=g, device=DEV) < OUTLIER_FRAC, x * OUTLIER_MUL, x)
        x = x.to(dt)
        return x.transpose(1, 2) if case["layout"] == "bshd" else x

    state = {"case": case, "q": tensor(Sq), "k": [tensor(L) for L in lens], "v": [tensor(L) for L in lens]}
    state["flags"] = usp.USP_ATTN_FUSED_PREFETCH if case["mode"] == "prefetch" else 0
    state["ks"] = state["vs"] = state["mask"] = None
    if case["kv"] == "fp8":   # what the chunks' owners have packed
        for t, s in (("k", "ks"), ("v", "vs")):
            packed = [usp.usp_fp8_quant(x.reshape(B * H * x.shape[2], d)) for x in state[t]]
            state[t] = [p[0].reshape(B, H, -1, d) for p in packed]
            state[s] = [p[1].reshape(B, H, -1) for p in packed]
    if case["masked"]:
        live = sum(lens) - case["masked"]
        keep = (torch.arange(sum(lens), device=DEV) < live).to(torch.uint8).expand(B, -1)
        state["mask"] = [m.contiguous() for m in keep.split(lens, dim=1)]
    state["out"] = torch.empty_like(state["q"])   # keeps a strided view's layout
    state["lse"] = torch.empty((B, H, Sq), device=DEV)
    desc = usp.make_attn_desc(state["q"], state["k"], state["out"], flags=state["flags"])
    need = usp.usp_ring_attn_workspace_bytes(desc)
    state["ws"] = torch.empty((need,), dtype=torch.uint8, device=DEV) if need else None
    return state


def run(state):
    op, s = state["case"]["op"], state
    if op == "payload":
        usp.usp_fp8_quant(s["x"], s["q"], s["s"])
        usp.usp_fp8_dequant(s["q"], s["s"], y=s["y"])
        return {"q": s["q"], "s": s["s"], "y": s["y"]}
    if op == "a2a":
        m = s["map"]
        usp.usp_fp8_quant_mapped(s["x"], m["n"], m["seq_sharded"], m["dense"], s["case"]["d"], s["q"], s["s"])
        usp.usp_fp8_dequant_mapped(s["q"], s["s"], m["n"], m["dense"], m["head_sharded"], s["y"])
        return {"q": s["q"], "s": s["s"], "y": s["y"]}
    if op == "merge":
        return usp.usp_lse_merge(s["o1"], s["l1"], s["o2"], s["l2"], s["o"], s["l"])
    return usp.usp_ring_attn_fwd(s["q"], s["k"], s["v"], k_scales=s["ks"], v_scales=s["vs"], key_mask=s["mask"],
                                 flags=s["flags"], out=s["out"], lse=s["lse"], workspace=s["ws"])


def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    if case["op"] == "payload":   # read x, write codes and scales; read them, write y
        return {"bytes": 2 * (case["rows"] * case["cols"] * (e + 1) + 4 * case["rows"]), "flops": 0}
    if case["op"] == "a2a":
        rows = case["B"] * case["H"] * case["S"]
        return {"bytes": 2 * (rows * case["d"] * (e + 1) + 4 * rows), "flops": 0}
    if case["op"] == "merge":
        return {"bytes": case["rows"] * (3 * case["d"] * e + 12), "flops": 0}
    live = (case["n"] - 1) * case["chunk"] + case["last"] - case["masked"]
    heads = case["B"] * case["H"]
    kv = case["d"] + 4 if case["kv"] == "fp8" else case["d"] * e
    return {"bytes": heads * (case["Sq"] * (2 * case["d"] * e + 4) + 2 * live * kv), "flops": 4.0 * heads * case["Sq"] * live * case["d"]}


def tolerance(case):
    if case["op"] in ("payload", "a2a"):
        return "exact"
    if case["op"] == "merge":
        # the rounding of the bf16 output alone is 1.7e-3 against 64 bits
        return {"rel": 4e-3} if case["dtype"] == "bf16" else {"rel": 1e-6}
    if case["dtype"] == "f32":   # 4e-7 to 6e-7 against the same path in 64 bits
        return {"rel": 4e-6}
    # head dimensions 64 and 128: P enters the second contraction as bf16 (2.5e-3 to 4.7e-3 between orders of the
    # sums, 2.4e-3 against 64 bits); the others keep fp32 up to the rounding of the output (1.7e-3 against 64 bits)
    return {"rel": 1e-2} if case["d"] in (64, 128) else {"rel": 4e-3}
