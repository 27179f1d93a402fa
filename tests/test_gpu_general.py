"""Attention outside the bf16 d = 128 / 64 kernels (attn_tile.h) against the fp64 oracle: both engines, every
size class of the head dimension and its edges, waves that share queries and waves that do not, ragged,
empty and masked chunks, FP8 K/V.  Bars: fp32 results 2e-5 / 5e-6 / 2e-5 as elsewhere; bf16 results carry
the rounding of the output plus the fp32 bar, because nothing inside is rounded to bf16: with 8 significant
bits a value in [2^e, 2^(e+1)) has neighbours 2^(e-7) apart, so rounding to nearest moves it by at most
2^(e-8), which is at most 2^-8 of the value.  That alone would let weights in bf16 pass, so the entries that
differ from the rounded oracle are counted too (BF16_MOVED)."""
import numpy as np
import pytest
import torch

from oracle import usp_oracle as orc
from paper_2602_10940_amd import workloads as W
from tests.gpu_util import BF16_MOVED, DEV, attn_errors, bf16_ulps, dev_bf16, dev_f32, host_bits_bf16, host_f64

pytestmark = pytest.mark.gpu

# B, H, d, Sq, chunks, masked keys, FP8 K/V
SHAPES = [
    (1, 1, 8, 1, (1,), (0, 0), False),                  # smallest
    (2, 3, 40, 77, (100, 0, 65), (90, 165), False),     # empty middle chunk, last chunk and a tail masked
    (1, 2, 64, 63, (64, 63), (0, 0), False),            # (bf16: the other kernels)
    (1, 3, 72, 130, (65, 128), (0, 64), False),         # first tile all dead
    (1, 2, 96, 64, (200,), (0, 0), False),
    (2, 2, 104, 33, (64, 64, 1), (0, 0), False),
    (1, 40, 80, 450, (129,), (0, 0), False),            # 64-query work-groups (waves do not share queries)
    (1, 40, 136, 450, (70,), (3, 9), False),
    (1, 2, 160, 50, (90,), (0, 0), False),
    (1, 3, 168, 20, (64, 10), (0, 0), False),
    (1, 2, 256, 65, (130,), (0, 0), False),
    (1, 40, 256, 260, (66,), (0, 0), False),
    (1, 3, 72, 40, (96, 33), (100, 129), True),         # rows of codes 8-byte aligned only
    (2, 20, 96, 300, (64, 65), (0, 0), True),
    (1, 2, 248, 17, (70,), (0, 0), True),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,H,d,Sq,lens,masked,fp8", SHAPES)
def test_general_shapes(dtype, B, H, d, Sq, lens, masked, fp8):
    import paper_2602_10940_amd as P
    wl = W.Workload("general", 500 + d, B, H, d, Sq, lens, dtype, masked_keys=masked)
    inp = W.make_attention_inputs(wl)
    up = dev_f32 if dtype == "f32" else dev_bf16
    kw = dict(key_mask=None if inp.key_mask is None else [torch.from_numpy(m).to(DEV) for m in inp.key_mask],
              softmax_scale=float(inp.softmax_scale))
    ks, vs, kx, vx = [up(k) for k in inp.k], [up(v) for v in inp.v], inp.k, inp.v
    if fp8:
        def pack(ts):
            qs = [P.usp_fp8_quant(t.reshape(-1, d)) for t in ts]
            return ([q.reshape(t.shape) for (q, _), t in zip(qs, ts)], [s.reshape(t.shape[:3]) for (_, s), t in zip(qs, ts)])
        (ks, ksc), (vs, vsc) = pack(ks), pack(vs)
        kw.update(k_scales=ksc, v_scales=vsc)
        kx = [orc.dequant_exact_f64(q.cpu().numpy(), s.cpu().numpy()) for q, s in zip(ks, ksc)]
        vx = [orc.dequant_exact_f64(q.cpu().numpy(), s.cpu().numpy()) for q, s in zip(vs, vsc)]
    o, l = P.usp_ring_attn_fwd(up(inp.q), ks, vs, **kw)
    torch.cuda.synchronize()
    ro, rl = orc.ring_attention(inp.q, kx, vx, float(inp.softmax_scale), inp.key_mask)
    got_o, got_l = host_f64(o), host_f64(l)
    mx, rel = attn_errors(got_o, ro)
    assert np.array_equal(np.isneginf(got_l), np.isneginf(rl))
    fin = np.isfinite(rl)
    if dtype == "bf16" and d == 64:
        assert mx <= 2e-2 and rel <= 5e-3 and np.max(np.abs(got_l - rl)[fin]) <= 1e-3
        return
    size = max(1.0, float(np.max(np.abs(ro))))
    out_max, out_rel = (0.0, 0.0) if dtype == "f32" else (2.0 ** -8 * size, 2.0 ** -8)
    assert mx <= 2e-5 * size + out_max and rel <= 5e-6 + out_rel and np.max(np.abs(got_l - rl)[fin], initial=0.0) <= 2e-5, (mx, rel)
    if dtype == "bf16":
        moved = np.count_nonzero(bf16_ulps(host_bits_bf16(o), ro))
        assert moved <= max(1, BF16_MOVED * ro.size), (moved, ro.size)
    # one launch over the chunks and a launch per chunk: the same operations, the same bits
    o2, l2 = P.usp_ring_attn_fwd(up(inp.q), ks, vs, flags=P.USP_ATTN_STEPWISE, **kw)
    torch.cuda.synchronize()
    assert torch.equal(o, o2) and torch.equal(l, l2)


@pytest.mark.parametrize("dtype,d", [("bf16", 72), ("f32", 64), ("bf16", 160)])
@pytest.mark.parametrize("lens", [(100, 65), (64, 64, 30)])
def test_strided_chunks_with_nothing_readable_behind_them(dtype, d, lens):
    """[B, S, H, d] storage of several chunks in one launch; the tokens behind each chunk's last one are NaN."""
    import paper_2602_10940_amd as P
    B, H, Sq, room = 2, 3, 70, 160
    inp = W.make_attention_inputs(W.Workload("strided", 90 + d, B, H, d, Sq, lens, dtype))
    up = dev_f32 if dtype == "f32" else dev_bf16

    def view(x):
        t = up(x)
        store = torch.full((B, room, H, d), float("nan"), dtype=t.dtype, device=DEV)
        store[:, :x.shape[2]] = t.transpose(1, 2)
        return store[:, :x.shape[2]].transpose(1, 2)
    q, scale = up(inp.q), float(inp.softmax_scale)
    o, l = P.usp_ring_attn_fwd(q, [view(k) for k in inp.k], [view(v) for v in inp.v], softmax_scale=scale)
    o2, l2 = P.usp_ring_attn_fwd(q, [up(k) for k in inp.k], [up(v) for v in inp.v], softmax_scale=scale)
    torch.cuda.synchronize()
    assert torch.equal(o, o2) and torch.equal(l, l2)
    ro, rl = orc.ring_attention(inp.q, inp.k, inp.v, scale)
    mx, rel = attn_errors(host_f64(o), ro)
    assert rel <= (5e-6 if dtype == "f32" else 2.0 ** -8) and np.max(np.abs(host_f64(l) - rl)) <= 2e-5


@pytest.mark.parametrize("dtype,d,Sq,H", [("bf16", 72, 20, 2), ("bf16", 72, 300, 60), ("f32", 64, 20, 2), ("f32", 64, 300, 60)])
def test_values_near_the_end_of_the_fp32_range(dtype, d, Sq, H):
    """|V| = 2e36 and scores that grow by less than 2^8 after the first tile: weights above 1 would take the sums
    (64 keys of up to 180 times 2e36) out of the fp32 range.  Every key has the same V, so that O is V."""
    import paper_2602_10940_amd as P
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    q = torch.zeros((1, H, Sq, d), dtype=dt, device=DEV)
    q[..., 0] = 1.0
    k = torch.zeros((1, H, 128, d), dtype=dt, device=DEV)
    k[:, :, 64:, 0] = 5.1875                                   # 2^7.48 with a scale of 1
    v = torch.full((1, H, 128, d), 2e36, dtype=dt, device=DEV)
    o, l = P.usp_ring_attn_fwd(q, [k], [v], softmax_scale=1.0)
    torch.cuda.synchronize()
    # 128 roundings of a sum at most; bf16: one rounding of the output on top
    tol = 128 * 2.0 ** -24 + (2.0 ** -8 if dtype == "bf16" else 0.0)
    assert float((o.double() / v[:, :, :1].double() - 1.0).abs().max()) <= tol
    assert float((l.double() - np.log(64.0 + 64.0 * np.exp(5.1875))).abs().max()) <= 2e-5


@pytest.mark.parametrize("dtype,B,H,d,Sq,lens", [("bf16", 2, 16, 72, 1024, (1024,)), ("bf16", 1, 4, 160, 300, (2000,)), ("f32", 2, 16, 32, 1000, (1000,)),
                                                 ("f32", 1, 8, 96, 700, (513, 513))])
def test_lse_is_as_exact_as_its_own_size_allows(dtype, B, H, d, Sq, lens):
    """lse = m ln 2 + log l with |lse| in [4, 16): the logarithm and the sum are rounded once each at the result's
    size or below (ulp 2^-21 to 8, 2^-20 beyond), and the scores, whose scale times log2 e is rounded once, move the
    result by 2^-24 of their weighted mean, here below 4: two units of the last place in all, per chunk."""
    import paper_2602_10940_amd as P
    g = torch.Generator(device=DEV)
    g.manual_seed(7)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    q = torch.randn((B, H, Sq, d), generator=g, device=DEV).to(dt)
    ks = [torch.randn((B, H, n, d), generator=g, device=DEV).to(dt) for n in lens]
    scale = float(np.float32(1.0 / np.sqrt(d)))
    _, l = P.usp_ring_attn_fwd(q, ks, ks, softmax_scale=scale)
    z = torch.matmul(q.double(), torch.cat(ks, 2).double().transpose(2, 3).contiguous()) * scale
    ref = torch.logsumexp(z, -1)
    ulp = torch.where(ref < 8.0, 2.0 ** -21, 2.0 ** -20)
    assert float(ref.min()) > 4.0 and float(ref.max()) < 16.0
    assert float(((l.double() - ref).abs() / ulp).max()) <= 2.0 * len(lens)


@pytest.mark.parametrize("d", [40, 64 + 8, 80, 96, 112, 120])
@pytest.mark.parametrize("H,Sq", [(2, 33), (60, 260), (60, 600)])   # few work-groups; 300 of 64 queries; 600 of them
def test_bf16_tiles_of_every_width(d, H, Sq):
    """Tiles that go to LDS directly, with eight and with four waves on a work-group's queries: columns past d, rows past
    the chunk, an empty chunk, dead keys, strided views with NaN behind them."""
    import paper_2602_10940_amd as P
    lens, room = (65, 0, 128), 140
    wl = W.Workload("widths", 300 + d, 1, H, d, Sq, lens, "bf16", masked_keys=(60, 120))
    inp = W.make_attention_inputs(wl)

    def view(x):
        t = dev_bf16(x)
        store = torch.full((1, room, H, d), float("nan"), dtype=t.dtype, device=DEV)
        store[:, :x.shape[2]] = t.transpose(1, 2)
        return store[:, :x.shape[2]].transpose(1, 2)
    km = [torch.from_numpy(m).to(DEV) for m in inp.key_mask]
    o, l = P.usp_ring_attn_fwd(dev_bf16(inp.q), [view(k) for k in inp.k], [view(v) for v in inp.v], key_mask=km, softmax_scale=float(inp.softmax_scale))
    torch.cuda.synchronize()
    ro, rl = orc.ring_attention(inp.q, inp.k, inp.v, float(inp.softmax_scale), inp.key_mask)
    mx, rel = attn_errors(host_f64(o), ro)
    size = max(1.0, float(np.max(np.abs(ro))))
    assert mx <= (2e-5 + 2.0 ** -8) * size and rel <= 5e-6 + 2.0 ** -8 and np.max(np.abs(host_f64(l) - rl)) <= 2e-5, (mx, rel)
    assert np.count_nonzero(bf16_ulps(host_bits_bf16(o), ro)) <= max(1, BF16_MOVED * ro.size)


@pytest.mark.parametrize("d,H,Sq", [(40, 3, 65), (56, 3, 65), (56, 60, 200), (72, 3, 65), (96, 3, 65), (96, 64, 128), (96, 43, 192), (112, 3, 65), (112, 60, 200)])
@pytest.mark.parametrize("masked", [None, (60, 120)])
def test_few_work_groups_through_registers_and_directly(d, H, Sq, masked):
    """Both ways a tile of few work-groups can come, at each width that has a rule, on both sides of d = 96's 128 work-groups."""
    import paper_2602_10940_amd as P
    wl = W.Workload("few", 500 + d, 1, H, d, Sq, (65, 0, 127), "bf16", **({"masked_keys": masked} if masked else {}))
    inp = W.make_attention_inputs(wl)
    km = None if masked is None else [torch.from_numpy(m).to(DEV) for m in inp.key_mask]
    o, l = P.usp_ring_attn_fwd(dev_bf16(inp.q), [dev_bf16(k) for k in inp.k], [dev_bf16(v) for v in inp.v], key_mask=km,
                               softmax_scale=float(inp.softmax_scale))
    torch.cuda.synchronize()
    ro, rl = orc.ring_attention(inp.q, inp.k, inp.v, float(inp.softmax_scale), inp.key_mask if masked else None)
    mx, rel = attn_errors(host_f64(o), ro)
    assert mx <= (2e-5 + 2.0 ** -8) * max(1.0, float(np.max(np.abs(ro)))) and rel <= 5e-6 + 2.0 ** -8 and np.max(np.abs(host_f64(l) - rl)) <= 2e-5, (mx, rel)
    assert np.count_nonzero(bf16_ulps(host_bits_bf16(o), ro)) <= max(1, BF16_MOVED * ro.size)


@pytest.mark.parametrize("d,H,Sq", [(72, 3, 40), (72, 60, 300), (160, 3, 40)])
@pytest.mark.parametrize("size", [12, 60, 100])
def test_fp8_values_with_scales_far_from_one(size, d, H, Sq):
    """V of 2^size in FP8: the weights come times scales of some 2^(size - 7) into the second product, split into bf16 parts there."""
    import paper_2602_10940_amd as P
    inp = W.make_attention_inputs(W.Workload("scaled", 40 + d, 1, H, d, Sq, (100, 65), "bf16"))

    def pack(ts):
        qs = [P.usp_fp8_quant(dev_f32(t).reshape(-1, d)) for t in ts]
        return [q.reshape(t.shape) for (q, _), t in zip(qs, ts)], [s.reshape(t.shape[:3]) for (_, s), t in zip(qs, ts)]
    (ks, ksc), (vs, vsc) = pack(inp.k), pack([np.ldexp(v, size).astype(np.float32) for v in inp.v])
    o, l = P.usp_ring_attn_fwd(dev_bf16(inp.q), ks, vs, k_scales=ksc, v_scales=vsc, softmax_scale=float(inp.softmax_scale))
    torch.cuda.synchronize()
    kx, vx = ([orc.dequant_exact_f64(q.cpu().numpy(), s.cpu().numpy()) for q, s in zip(a, b)] for a, b in ((ks, ksc), (vs, vsc)))
    ro, rl = orc.ring_attention(inp.q, kx, [np.ldexp(v, -size) for v in vx], float(inp.softmax_scale))
    got = np.ldexp(host_f64(o), -size)
    mx, rel = attn_errors(got, ro)
    assert mx <= (2e-5 + 2.0 ** -8) * max(1.0, float(np.max(np.abs(ro)))) and rel <= 5e-6 + 2.0 ** -8 and np.max(np.abs(host_f64(l) - rl)) <= 2e-5, (mx, rel)
    assert np.count_nonzero(bf16_ulps(host_bits_bf16(o), np.ldexp(ro, size))) <= max(1, BF16_MOVED * ro.size)


# B, H, d, Sq, keys, (first masked, last masked + 1), FP8 K/V
SHARED = [
    ("f32", 1, 2, 8, 17, 704, (0, 0), False),            # eleven tiles, two to three a work-group
    ("f32", 1, 3, 64, 100, 1025, (0, 0), False),         # the last work-group's range ends in a tile of one key
    ("f32", 2, 2, 104, 16, 1000, (0, 600), False),       # work-groups without a live key
    ("f32", 1, 1, 128, 1, 2000, (0, 2000), False),       # no live key at all
    ("f32", 1, 2, 72, 33, 1100, (700, 1100), True),
    ("bf16", 1, 2, 40, 33, 1025, (1, 1024), False),      # the first and the last key live
    ("bf16", 2, 4, 72, 100, 1549, (0, 0), False),
    ("bf16", 1, 2, 96, 64, 769, (0, 0), False),
    ("bf16", 1, 2, 136, 31, 1100, (500, 777), False),
    ("bf16", 1, 2, 160, 65, 1280, (0, 0), True),
    ("bf16", 2, 3, 72, 20, 1200, (0, 300), True),
]


@pytest.mark.parametrize("dtype,B,H,d,Sq,keys,masked,fp8", SHARED)
def test_work_groups_that_share_the_keys_of_a_query_block(dtype, B, H, d, Sq, keys, masked, fp8):
    """Against the oracle (bars as above) and against the same call without the workspace, which one work-group per query block
    serves: with room for the shares, with too little, through the entry point that uses none, and replayed from a graph; inputs and result in [B, S, H, d] storage."""
    import paper_2602_10940_amd as P
    inp = W.make_attention_inputs(W.Workload("shared", 700 + d, B, H, d, Sq, (keys,), dtype, masked_keys=masked))
    up = dev_f32 if dtype == "f32" else dev_bf16
    bshd = lambda t: t.transpose(1, 2).contiguous().transpose(1, 2)
    q, k, v, scale = bshd(up(inp.q)), bshd(up(inp.k[0])), bshd(up(inp.v[0])), float(inp.softmax_scale)
    kw = dict(softmax_scale=scale, key_mask=None if inp.key_mask is None else [torch.from_numpy(m).to(DEV) for m in inp.key_mask])
    kx, vx = inp.k[0], inp.v[0]
    if fp8:
        (k, ksc), (v, vsc) = [P.usp_fp8_quant(t.contiguous().reshape(-1, d)) for t in (k, v)]
        k, v = k.reshape(B, H, keys, d), v.reshape(B, H, keys, d)
        kw.update(k_scales=[ksc.reshape(B, H, keys)], v_scales=[vsc.reshape(B, H, keys)])
        kx, vx = [orc.dequant_exact_f64(c.cpu().numpy(), s.cpu().numpy().reshape(B, H, keys)) for c, s in ((k, ksc), (v, vsc))]
    room = torch.empty((B, Sq, H, d), dtype=q.dtype, device=DEV).transpose(1, 2)
    need = P.usp_ring_attn_workspace_bytes(P.make_attn_desc(q, [k], room, flags=0))
    assert need >= 2 * B * H * Sq * (d + 2) * 4     # shared by two work-groups at least
    run = lambda **more: P.usp_ring_attn_fwd(q, [k], [v], **kw, **more)
    o, l = run(out=room)
    small, small_l = run(workspace=torch.empty(256, dtype=torch.uint8, device=DEV))
    go, gl = torch.empty_like(q), torch.empty((B, H, Sq), dtype=torch.float32, device=DEV)
    P.usp_ring_attn_fwd_noalloc(q, [k], [v], go, gl, **kw)
    assert torch.equal(go, small) and torch.equal(gl, small_l)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(out=go, lse=gl, workspace=ws)
    for _ in range(3):
        ws.fill_(255)                               # (NaN)
        go.zero_(), gl.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(go, o) and torch.equal(gl, l)
    ro, rl = orc.ring_attention(inp.q, [kx], [vx], scale, inp.key_mask)
    for x, y in ((o, l), (small, small_l)):
        got_o, got_l = host_f64(x), host_f64(y)
        mx, rel = attn_errors(got_o, ro)
        fin = np.isfinite(rl)
        size = max(1.0, float(np.max(np.abs(ro))))
        out_max, out_rel = (0.0, 0.0) if dtype == "f32" else (2.0 ** -8 * size, 2.0 ** -8)
        assert mx <= 2e-5 * size + out_max and rel <= 5e-6 + out_rel, (mx, rel)
        assert np.array_equal(np.isneginf(got_l), np.isneginf(rl)) and np.max(np.abs(got_l[fin] - rl[fin]), initial=0.0) <= 2e-5
        if dtype == "bf16":
            assert np.count_nonzero(bf16_ulps(host_bits_bf16(x), ro)) <= max(1, BF16_MOVED * ro.size)


def test_the_workspace_of_a_call_belongs_to_the_stream_it_runs_on():
    import paper_2602_10940_amd as P
    q = torch.zeros((1, 2, 100, 72), dtype=torch.bfloat16, device=DEV)
    k = torch.zeros((1, 2, 1549, 72), dtype=torch.bfloat16, device=DEV)
    out, lse = torch.empty_like(q), torch.empty((1, 2, 100), dtype=torch.float32, device=DEV)
    torch.cuda.synchronize()
    st, before = torch.cuda.Stream(), torch.cuda.current_stream()
    P.usp_ring_attn_fwd(q, [k], [k], out=out, lse=lse, compute_stream=st)
    assert torch.cuda.current_stream() == before
    at, size = out._usp_workspace.data_ptr(), out._usp_workspace.numel()
    out._usp_workspace = None
    other = torch.empty(size, dtype=torch.uint8, device=DEV)      # memory of the current stream
    with torch.cuda.stream(st):
        again = torch.empty(size, dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    assert again.data_ptr() == at and other.data_ptr() != at
