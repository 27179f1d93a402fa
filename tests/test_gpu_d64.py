"""bf16 attention with head dimension 64: the call runs on the matrix-core kernels in their
head-dimension-64 form (128-byte rows of Q, K, V and O read and written in place).  Parity against the
fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import usp_oracle as orc
from paper_2602_10940_amd import workloads as W
from tests.gpu_util import DEV, dev_bf16, host_f64
from tests.test_gpu_attention import _assert_parity, _oracle, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,Sq,lens,flags", [
    (1, 3, 200, (192, 100), 0),            # a ragged chunk: one launch per chunk with key records
    (2, 2, 300, (128, 256, 64), 0),        # whole tiles: one launch over the ring
    (1, 2, 130, (128, 256, 64), 16),       # ... with the transfers inside
    (1, 2, 130, (136,) * 3, 1),            # side-stream double buffering
    (1, 4, 520, (320,), 4),                # one chunk, 256-query work-groups
    (1, 2, 150, (200, 136), 2),            # merge as a separate kernel
    (1, 36, 2048, (128,), 0),              # 288 query blocks: d = 128 would take the mixed launch here
    (1, 3, 300, (128, 64), 32),            # the mixed launch asked for by flag
])
def test_bf16_d64_against_oracle(B, H, Sq, lens, flags):
    wl = W.Workload("d64", 91, B, H, 64, Sq, tuple(lens), "bf16")
    inp = W.make_attention_inputs(wl)
    side = torch.cuda.Stream() if flags == 1 else None
    o, l = _run(inp, flags=flags, copy_stream=side)
    assert o.shape == (B, H, Sq, 64)
    ro, rl = _oracle(inp)
    _assert_parity(o, l, ro, rl)


def test_bf16_d64_with_key_mask_and_strided_layout():
    """[B,S,H,d] storage viewed as [B,H,S,d] for Q, K, V and O, and a key mask over the second chunk."""
    import paper_2602_10940_amd as P
    wl = W.Workload("d64_masked", 92, 2, 3, 64, 140, (200, 136), "bf16", masked_keys=(300, 336))
    inp = W.make_attention_inputs(wl)
    ro, rl = _oracle(inp)
    o, l = _run(inp)
    _assert_parity(o, l, ro, rl)
    whole_k = np.concatenate(inp.k, axis=2); whole_v = np.concatenate(inp.v, axis=2)
    def bshd(x):
        return dev_bf16(np.ascontiguousarray(x.transpose(0, 2, 1, 3))).permute(0, 2, 1, 3)
    q, kk, vv = bshd(inp.q), bshd(whole_k), bshd(whole_v)
    ks = [kk[:, :, :200], kk[:, :, 200:]]; vs = [vv[:, :, :200], vv[:, :, 200:]]
    out = torch.empty((2, 140, 3, 64), dtype=torch.bfloat16, device=DEV).permute(0, 2, 1, 3)
    km = [torch.from_numpy(m).to(DEV) for m in inp.key_mask]
    o2, l2 = P.usp_ring_attn_fwd(q, ks, vs, key_mask=km, softmax_scale=float(inp.softmax_scale), out=out)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(host_f64(o2), o)
    np.testing.assert_array_equal(host_f64(l2), l)


def test_bf16_d64_default_scale_is_that_of_the_original_head_dimension():
    import paper_2602_10940_amd as P
    wl = W.Workload("d64_scale", 93, 1, 2, 64, 100, (128,), "bf16")
    inp = W.make_attention_inputs(wl)
    q = dev_bf16(inp.q); k = dev_bf16(inp.k[0]); v = dev_bf16(inp.v[0])
    o0, l0 = P.usp_ring_attn_fwd(q, [k], [v], softmax_scale=0.0)       # 0: the library's 1 / sqrt(d)
    o1, l1 = P.usp_ring_attn_fwd(q, [k], [v], softmax_scale=0.125)
    torch.cuda.synchronize()
    assert torch.equal(o0, o1) and torch.equal(l0, l1)
    ro, rl = orc.ring_attention(inp.q, inp.k, inp.v, 0.125)
    _assert_parity(host_f64(o0), host_f64(l0), ro, rl)


@pytest.mark.parametrize("lens,flags", [((192, 100), 0), ((128, 256, 64), 0), ((128, 256, 64), 64), ((128, 192), 16),
                                        ((256, 0), 0), ((256, 64, 0), 1), ((0, 128, 0, 64), 16)])   # empty chunks, also last
def test_fp8_kv_d64_ring_against_oracle(lens, flags):
    """FP8 K/V chunks with d = 64 (ragged chunks: one launch per chunk; whole tiles: the one-launch
    form with the decode inside), a key mask over the tail."""
    import paper_2602_10940_amd as P
    S = sum(lens)
    wl = W.Workload("d64_fp8", 94, 2, 3, 64, 150, tuple(lens), "bf16", masked_keys=(S - 40, S))
    inp = W.make_attention_inputs(wl)
    q = dev_bf16(inp.q)
    kq, ksc, vq, vsc, kx, vx = [], [], [], [], [], []
    for k, v in zip(inp.k, inp.v):
        B, H, L, d = k.shape
        if L == 0:
            kq.append(torch.empty((B, H, 0, d), dtype=torch.uint8, device=DEV)); vq.append(kq[-1])
            ksc.append(torch.empty((B, H, 0), dtype=torch.float32, device=DEV)); vsc.append(ksc[-1])
            kx.append(k.astype(np.float64)); vx.append(v.astype(np.float64))
            continue
        a, sa = P.usp_fp8_quant(dev_bf16(k).reshape(B * H * L, d))
        b, sb = P.usp_fp8_quant(dev_bf16(v).reshape(B * H * L, d))
        kq.append(a.reshape(B, H, L, d)); ksc.append(sa.reshape(B, H, L))
        vq.append(b.reshape(B, H, L, d)); vsc.append(sb.reshape(B, H, L))
        kx.append(orc.dequant_exact_f64(a.cpu().numpy().reshape(B, H, L, d), sa.cpu().numpy().reshape(B, H, L)))
        vx.append(orc.dequant_exact_f64(b.cpu().numpy().reshape(B, H, L, d), sb.cpu().numpy().reshape(B, H, L)))
    km = [torch.from_numpy(m).to(DEV) for m in inp.key_mask]
    o, l = P.usp_ring_attn_fwd(q, kq, vq, k_scales=ksc, v_scales=vsc, key_mask=km, softmax_scale=float(inp.softmax_scale),
                               flags=flags, copy_stream=torch.cuda.Stream() if flags & 1 else None)
    torch.cuda.synchronize()
    ro, rl = orc.ring_attention(inp.q, kx, vx, float(inp.softmax_scale), inp.key_mask)
    _assert_parity(host_f64(o), host_f64(l), ro, rl)


@pytest.mark.parametrize("H,Sq,keys,masked,fp8,split", [
    (26, 1300, 640, (0, 0), False, False),     # 286 blocks of 128, two to a CU: ten tiles are too few
    (26, 1300, 769, (0, 0), False, True),      # thirteen, the last one ragged
    (26, 1300, 768, (100, 300), False, True),  # dead tiles in the middle
    (64, 1024, 64, (0, 0), False, False),      # 512 blocks, one tile
    (27, 2400, 128, (0, 0), False, True),      # 513: the third work-group of a CU has it alone
    (26, 1300, 1024, (0, 0), True, False),     # from FP8 the line lies higher
    (27, 2400, 448, (0, 0), True, True),
    (27, 2400, 449, (0, 0), True, False),      # FP8 with dead keys: one work-group to a CU, the rule it had
    (26, 1300, 3136, (0, 0), True, False),     # and above what a call over whole tiles reaches while the chip takes all work-groups at once
    (27, 2400, 192, (0, 0), True, True),       # a round less: few tiles are enough
])
def test_d64_two_work_groups_to_a_cu(H, Sq, keys, masked, fp8, split):
    """The form that the rule picks over one chunk, as its flag gives it, against the oracle."""
    import paper_2602_10940_amd as P
    inp = W.make_attention_inputs(W.Workload("d64_two", 95, 1, H, 64, Sq, (keys,), "bf16", masked_keys=masked))
    q, k, v = dev_bf16(inp.q), dev_bf16(inp.k[0]), dev_bf16(inp.v[0])
    kw = {}
    kx, vx = inp.k[0], inp.v[0]
    if fp8:
        (a, sa), (b, sb) = (P.usp_fp8_quant(x.reshape(H * keys, 64)) for x in (k, v))
        kx, vx = (orc.dequant_exact_f64(c.cpu().numpy().reshape(1, H, keys, 64), s.cpu().numpy().reshape(1, H, keys)) for c, s in ((a, sa), (b, sb)))
        k, v = a.reshape(1, H, keys, 64), b.reshape(1, H, keys, 64)
        kw = {"k_scales": [sa.reshape(1, H, keys)], "v_scales": [sb.reshape(1, H, keys)]}
    if masked[1]:
        kw["key_mask"] = [torch.from_numpy(inp.key_mask[0]).to(DEV)]
    scale = float(inp.softmax_scale)
    o, l = P.usp_ring_attn_fwd(q, [k], [v], softmax_scale=scale, **kw)
    os_, ls = P.usp_ring_attn_fwd(q, [k], [v], softmax_scale=scale, flags=P.USP_ATTN_KERNEL_SPLIT, **kw)
    ow, lw = P.usp_ring_attn_fwd(q, [k], [v], softmax_scale=scale, flags=P.USP_ATTN_KERNEL_WIDE, **kw)
    torch.cuda.synchronize()
    same, other = ((os_, ls), ow) if split else ((ow, lw), os_)
    assert torch.equal(o, same[0]) and torch.equal(l, same[1])
    assert keys == 64 or not torch.equal(o, other)      # (one tile: there is nothing to divide)
    heads = [0, H - 1]
    ro, rl = orc.ring_attention(inp.q[:, heads], [kx[:, heads]], [vx[:, heads]], scale, inp.key_mask if masked[1] else None)
    for x, y in ((o, l), (os_, ls), (ow, lw)):
        _assert_parity(host_f64(x[:, heads]), host_f64(y[:, heads]), ro, rl)


@pytest.mark.parametrize("H,Sq,lens,masked,split", [
    (65, 1025, (64, 64), (0, 0), False),          # 325 blocks of 256, 585 of 128: two rounds, three work-groups to a CU
    (65, 1025, (192, 192), (0, 0), True),
    (65, 1025, (128, 320), (100, 300), True),     # dead tiles in the middle
    (65, 1025, (320, 321), (0, 0), True),         # ragged
    (26, 4096, (320, 320), (0, 0), False),        # 416 and 832: two rounds, four to a CU, few tiles
    (26, 4096, (1024, 1024), (0, 0), True),
    (300, 100, (64, 64), (0, 0), True),           # one round of pairs
])
def test_d64_rings_above_one_round(H, Sq, lens, masked, split):
    """The form that the rule picks, as its flag gives it, the chunks at hand and with the transfers inside, against the oracle."""
    import paper_2602_10940_amd as P
    inp = W.make_attention_inputs(W.Workload("d64_rounds", 97, 1, H, 64, Sq, lens, "bf16", masked_keys=masked))
    q, k, v = dev_bf16(inp.q), [dev_bf16(x) for x in inp.k], [dev_bf16(x) for x in inp.v]
    scale = float(inp.softmax_scale)
    kw = {"key_mask": [torch.from_numpy(x).to(DEV) for x in inp.key_mask]} if masked[1] else {}
    forms = P.USP_ATTN_KERNEL_WIDE, P.USP_ATTN_KERNEL_SPLIT
    got = [P.usp_ring_attn_fwd(q, k, v, softmax_scale=scale, flags=f, **kw) for f in (0, P.USP_ATTN_FUSED_PREFETCH, *forms)]
    torch.cuda.synchronize()
    (o, l), (op, lp), same, other = got[0], got[1], got[2 + split], got[3 - split]
    assert torch.equal(o, same[0]) and torch.equal(l, same[1]) and not torch.equal(o, other[0])
    assert torch.equal(o, op) and torch.equal(l, lp)
    heads = [0, H - 1]
    ro, rl = orc.ring_attention(inp.q[:, heads], [x[:, heads] for x in inp.k], [x[:, heads] for x in inp.v], scale, inp.key_mask if masked[1] else None)
    for x, y in (got[0], other):
        _assert_parity(host_f64(x[:, heads]), host_f64(y[:, heads]), ro, rl)


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("lens", [(64,), (128,), (1088,), (64, 192), (320, 64, 576)])
def test_d64_256_query_form_with_a_mask_that_masks_nothing(lens, fp8):
    """The form for dead keys, whose tiles lie otherwise in LDS (V's rows whole, from FP8), gives the bits of the one for none."""
    import paper_2602_10940_amd as P
    B, H, Sq = 2, 3, 530
    g = torch.Generator(device=DEV)
    g.manual_seed(sum(lens))
    q, *kv = (torch.randn((B, H, s, 64), generator=g, device=DEV).bfloat16() for s in (Sq,) + lens + lens)
    k, v, kw = kv[:len(lens)], kv[len(lens):], {}
    if fp8:
        ks, vs = ([P.usp_fp8_quant(x.reshape(-1, 64)) for x in y] for y in (k, v))
        k, v = ([c.reshape(B, H, -1, 64) for c, _ in y] for y in (ks, vs))
        kw = {"k_scales": [s.reshape(B, H, -1) for _, s in ks], "v_scales": [s.reshape(B, H, -1) for _, s in vs]}
    flags = P.USP_ATTN_KERNEL_WIDE
    o, l = P.usp_ring_attn_fwd(q, k, v, flags=flags, **kw)
    om, lm = P.usp_ring_attn_fwd(q, k, v, flags=flags, key_mask=[torch.ones((B, n), dtype=torch.uint8, device=DEV) for n in lens], **kw)
    assert torch.isfinite(o.float()).all() and torch.equal(o, om) and torch.equal(l, lm)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,Sq,keys,masked", [(1, 100, 1024, (0, 0)),         # (100 rows: the last work-group of the second launch half full)
                                              (1, 257, 4000, (0, 0)), (2, 33, 4096, (64, 2100)), (3, 130, 960, (959, 960)), (1, 7, 16384, (0, 0))])
def test_parts_put_together_against_oracle(d, H, Sq, keys, masked):
    """Two to sixteen parts, the second launch with fewer parts than it has room for, and parts without a live key."""
    from paper_2602_10940_amd import diag
    import paper_2602_10940_amd as P
    inp = W.make_attention_inputs(W.Workload("parts", 96, 1, H, d, Sq, (keys,), "bf16", masked_keys=masked))
    q, k = dev_bf16(inp.q), dev_bf16(inp.k[0])
    assert diag.usp_diag_attn_route(P.make_attn_desc(q, [k], torch.empty_like(q)), bool(masked[1])).parts > 1
    o, l = _run(inp)
    ro, rl = _oracle(inp)
    _assert_parity(o, l, ro, rl)
