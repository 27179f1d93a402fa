"""The ends of a matrix-core attention launch: rows that do not fill a wave, a work-group or a store instruction, in every
form that finishes or carries rows, and references of the exponent that lag the scores or stand far above them when the
halves of a work-group's keys are put together.  Parity against the fp64 oracle."""
import numpy as np
import pytest
import torch

from oracle import usp_oracle as orc
from paper_2602_10940_amd import workloads as W
from tests.gpu_util import DEV, dev_bf16, host_f64
from tests.test_gpu_attention import _assert_parity, _oracle

pytestmark = pytest.mark.gpu

WIDE, SPLIT, STEPWISE = 4, 8, 64


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("flags,lens", [
    (WIDE, (128,)), (SPLIT, (192,)),                              # a launch that writes the result
    (WIDE | STEPWISE, (64, 128, 64)), (SPLIT | STEPWISE, (64, 128, 64)),   # the carried state: first, middle, last chunk
    (0, (1088,)),                                                 # few work-groups: keys shared between them
])
@pytest.mark.parametrize("Sq", [1, 15, 17, 33, 129, 257])
def test_rows_at_the_ends(Sq, flags, lens, d):
    import paper_2602_10940_amd as P
    wl = W.Workload("ends", 17, 1, 3, d, Sq, lens, "bf16")
    inp = W.make_attention_inputs(wl)
    room = torch.full((1, 3, Sq + 5, d), 7.0, dtype=torch.bfloat16, device=DEV)   # rows behind the last stay what they are
    out, lse = P.usp_ring_attn_fwd(dev_bf16(inp.q), [dev_bf16(k) for k in inp.k], [dev_bf16(v) for v in inp.v],
                                   softmax_scale=float(inp.softmax_scale), flags=flags, out=room[:, :, :Sq])
    torch.cuda.synchronize()
    ro, rl = _oracle(inp)
    _assert_parity(host_f64(out), host_f64(lse), ro, rl)
    assert bool((room[:, :, Sq:] == 7.0).all())


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("flags", [WIDE, SPLIT, 0])
@pytest.mark.parametrize("levels", [
    (0, 62, 64, 66), (66, 64, 62, 0),               # 2^90 above the first maximum without a new reference, then past it
    (0, 62, 66, 66, 120, 62, 130, 131, 100),        # a second and a third move
    (0, 100, 62, 100, 0, 101, 62, 0),               # the two halves of the keys apart: one lags, the other has moved
    (40, 0, 39, 130, 41, 131, 127, 128, 129, 60),
])
def test_references_that_lag(levels, flags, d):
    """Scores that climb from tile to tile: what was summed before a reference moved may be all but the whole result."""
    import paper_2602_10940_amd as P
    rng = np.random.default_rng(5)
    n = 64 * len(levels)
    q = np.zeros((1, 2, 40, d), np.float32)
    q[..., 0] = rng.choice([1.0, 0.75, 0.5], size=(1, 2, 40))
    k = np.zeros((1, 2, n, d), np.float32)
    k[..., 0] = np.repeat(np.asarray(levels, np.float32), 64) - rng.integers(0, 8, size=(1, 2, n)) * 0.5   # bf16 holds these
    v = W.bf16_bits_to_f32(W.f32_to_bf16_bits(rng.standard_normal((1, 2, n, d)).astype(np.float32))).reshape(1, 2, n, d)
    kb = W.bf16_bits_to_f32(W.f32_to_bf16_bits(k)).reshape(k.shape)
    out, lse = P.usp_ring_attn_fwd(dev_bf16(q), [dev_bf16(kb)], [dev_bf16(v)], softmax_scale=1.0, flags=flags)
    torch.cuda.synchronize()
    ro, rl = orc.ring_attention(q, [kb], [v], 1.0, None)
    _assert_parity(host_f64(out), host_f64(lse), ro, rl)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("flags", [WIDE, SPLIT, 0, WIDE | STEPWISE])
@pytest.mark.parametrize("size", [0, -60, -76, -84, -92])
def test_small_values_under_outgrown_references(size, flags, d):
    """V of 2^size beside scores whose references have been outgrown: a weight is at least 2^-32 of one where it counts, so
    that the smallest of these products, 2^-124, is a normal number of fp32 and O as exact as for V of order one."""
    import paper_2602_10940_amd as P
    rng = np.random.default_rng(6)
    levels = (0, 0, 100, 100, 62, 62, 99, 99, 20, 20)          # in pairs of tiles: both halves of the keys outgrow theirs
    n = 64 * len(levels)
    q = np.zeros((1, 2, 40, d), np.float32)
    q[..., 0] = rng.choice([1.0, 0.984375, 0.96875], size=q.shape[:3])
    k = np.zeros((1, 2, n, d), np.float32)
    k[..., 0] = np.repeat(np.asarray(levels, np.float32), 64) - rng.integers(0, 8, size=(1, 2, n)) * 0.5   # bf16 holds these
    v = W.bf16_bits_to_f32(W.f32_to_bf16_bits(rng.standard_normal((1, 2, n, d)).astype(np.float32))).reshape(k.shape)
    small = np.ldexp(v, size).astype(np.float32)              # (exact: bf16 holds them)
    lens = (192, 256, 192) if flags & STEPWISE else (n,)
    cut = np.cumsum((0,) + lens)
    kd, vd = ([dev_bf16(np.ascontiguousarray(x[:, :, a:b])) for a, b in zip(cut, cut[1:])] for x in (k, small))
    out, lse = P.usp_ring_attn_fwd(dev_bf16(q), kd, vd, softmax_scale=1.0, flags=flags)
    torch.cuda.synchronize()
    _assert_parity(np.ldexp(host_f64(out), -size), host_f64(lse), *orc.ring_attention(q, [k], [v], 1.0, None))


def _bf16(x):
    return W.bf16_bits_to_f32(W.f32_to_bf16_bits(np.asarray(x, np.float32))).reshape(np.shape(x))


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("flags", [WIDE, SPLIT, 0, WIDE | STEPWISE, SPLIT | STEPWISE])
@pytest.mark.parametrize("at", [320, 364, 384, 447])
def test_one_key_is_the_row(at, flags, d):
    """Once a reference has been outgrown, a row that is one key's (all others count less than e^-25 together) is that key's
    V to the bit: weight over sum of weights is 1 to fp32 rounding, however the weight itself was rounded.  The weight lies
    just beside the middle between two bf16 values, so that O over the sum of the unrounded weights would be another bf16
    value for most of V, which is checked here.  (Key-split: the key is in the sixth or the seventh tile, and its half of the
    keys has outgrown a reference two tiles ahead of it.)"""
    import paper_2602_10940_amd as P
    rng = np.random.default_rng(at)
    tiles = (0, 0, 0, 100, 100, 100, 100)
    n = 64 * len(tiles)
    q = np.zeros((1, 2, 40, d), np.float32)
    k = np.zeros((1, 2, n, d), np.float32)
    k[..., 0] = np.repeat(np.asarray(tiles, np.float32), 64)
    k[:, :, at, 0] = 140.0
    k[:, :, at, 1:3] = 1.0
    # the key's exponent above the others', (40 q0 + q1 + q2) log2 e, is a whole number and the log2 of the weight's mantissa
    q[..., 0] = rng.choice([1.0, 0.984375, 0.96875, 0.953125], size=(1, 2, 40))
    mantissa = rng.choice([1.0033, 1.0045], size=(1, 2, 40))                    # (1.00390625 lies between 1 and 1.0078125)
    up = q[..., 0].astype(np.float64) * 40 * np.log2(np.e)
    left = (np.floor(up) + 1 + np.log2(mantissa) - up) / np.log2(np.e)
    q[..., 1] = _bf16(left)
    q[..., 2] = _bf16(left - q[..., 1])
    v = _bf16(rng.standard_normal((1, 2, n, d)))
    p = np.exp2(((q[..., 0].astype(np.float64) * 40 + q[..., 1] + q[..., 2]) * np.log2(np.e)) % 1.0)[..., None]
    row = v[:, :, at:at + 1].astype(np.float64)
    assert np.abs(p[..., 0] - mantissa).max() < 1e-4 and np.mean(_bf16(_bf16(p) * row / p) != row) > 0.5
    lens = (64, 384) if flags & STEPWISE else (n,)
    cut = np.cumsum((0,) + lens)
    kd, vd = ([dev_bf16(np.ascontiguousarray(x[:, :, a:b])) for a, b in zip(cut, cut[1:])] for x in (k, v))
    out, lse = P.usp_ring_attn_fwd(dev_bf16(q), kd, vd, softmax_scale=1.0, flags=flags)
    torch.cuda.synchronize()
    assert np.array_equal(host_f64(out), np.broadcast_to(row, q.shape))
    _assert_parity(host_f64(out), host_f64(lse), *orc.ring_attention(q, [k], [v], 1.0, None))


def _rows_of(which):
    """Of 40 queries, those of the first, the second or both blocks of sixteen that a wave holds."""
    block = np.arange(40) // 16 % 2
    return np.ones(40, bool) if which == "both" else block == (which == "second")


def _from_fp8(x):
    """Codes and scales on the GPU, and the values they stand for, float64."""
    import paper_2602_10940_amd as P
    c, s = P.usp_fp8_quant(dev_bf16(x).reshape(-1, x.shape[-1]))
    return c.reshape(x.shape), s.reshape(x.shape[:3]), orc.dequant_exact_f64(c.cpu().numpy().reshape(x.shape), s.cpu().numpy().reshape(x.shape[:3]))


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("flags", [WIDE, SPLIT])
@pytest.mark.parametrize("which", ["first", "second", "both"])
@pytest.mark.parametrize("levels", [(0, 62, 64, 66), (0, 62, 66, 66, 120, 62, 130, 131, 100), (0, 100, 62, 100, 0, 101, 62, 0)])
def test_references_that_lag_from_fp8(levels, which, flags, d):
    """Whole unmasked tiles from FP8, where the key-split form of d = 64 certifies one block of sixteen queries after the other: the scores of
    one block, of the other or of both climb, those of the rest stay 0."""
    import paper_2602_10940_amd as P
    rng = np.random.default_rng(7)
    n = 64 * len(levels)
    q = np.zeros((1, 2, 40, d), np.float32)
    q[..., 0] = rng.choice([1.0, 0.75, 0.5], size=(1, 2, 40)) * _rows_of(which)
    k = np.zeros((1, 2, n, d), np.float32)
    k[..., 0] = np.repeat(np.asarray(levels, np.float32), 64) - rng.integers(0, 8, size=(1, 2, n)) * 0.5
    kc, ks, kx = _from_fp8(k)
    vc, vs, vx = _from_fp8(_bf16(rng.standard_normal((1, 2, n, d))))
    out, lse = P.usp_ring_attn_fwd(dev_bf16(q), [kc], [vc], k_scales=[ks], v_scales=[vs], softmax_scale=1.0, flags=flags)
    torch.cuda.synchronize()
    _assert_parity(host_f64(out), host_f64(lse), *orc.ring_attention(q, [kx], [vx], 1.0, None))


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("flags", [WIDE, SPLIT])
@pytest.mark.parametrize("which", ["first", "second", "both"])
@pytest.mark.parametrize("at", [320, 447])
def test_one_key_is_the_row_from_fp8(at, which, flags, d):
    """As test_one_key_is_the_row, for the queries of one block or of both."""
    import paper_2602_10940_amd as P
    rng = np.random.default_rng(at)
    n = 64 * 7
    rows = _rows_of(which)
    k = np.zeros((1, 2, n, d), np.float32)
    k[:, :, 192:, 0] = 100.0
    k[:, :, at, 0] = 140.0
    k[:, :, at, 1:3] = 1.0
    kc, ks, kx = _from_fp8(k)
    k0, k1, rest = kx[0, 0, at, 0], kx[0, 0, at, 1], kx[0, 0, -1 if at != n - 1 else -2, 0]
    assert k0 == 140.0 and 0.9 < k1 < 1.1 and abs(rest - 100.0) < 1e-4
    q = np.zeros((1, 2, 40, d), np.float32)
    q[..., 0] = rng.choice([1.0, 0.984375, 0.96875, 0.953125], size=(1, 2, 40)) * rows
    mantissa = rng.choice([1.0033, 1.0045], size=(1, 2, 40))
    up = q[..., 0].astype(np.float64) * 40 * np.log2(np.e)
    left = (np.floor(up) + 1 + np.log2(mantissa) - up) / np.log2(np.e) / k1 * rows
    q[..., 1] = _bf16(left)
    q[..., 2] = _bf16(left - q[..., 1])
    vc, vs, vx = _from_fp8(_bf16(rng.standard_normal((1, 2, n, d))))
    row = _bf16((vc[:, :, at:at + 1].view(torch.float8_e4m3fn).float() * vs[:, :, at:at + 1, None]).cpu().numpy()).astype(np.float64)
    p = np.exp2(((q[..., 0].astype(np.float64) * 40 + k1 * (q[..., 1].astype(np.float64) + q[..., 2])) * np.log2(np.e)) % 1.0)[..., None]
    assert np.abs(p[:, :, rows, 0] - mantissa[:, :, rows]).max() < 1e-4 and np.mean((_bf16(_bf16(p) * row / p) != row)[:, :, rows]) > 0.5
    out, lse = P.usp_ring_attn_fwd(dev_bf16(q), [kc], [vc], k_scales=[ks], v_scales=[vs], softmax_scale=1.0, flags=flags)
    torch.cuda.synchronize()
    assert np.array_equal(host_f64(out)[:, :, rows], np.broadcast_to(row, q.shape)[:, :, rows])
    _assert_parity(host_f64(out), host_f64(lse), *orc.ring_attention(q, [kx], [vx], 1.0, None))


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("H,lens", [(1, (64, 64)), (1, (640, 1)), (3, (321, 319, 322)), (5, (128, 192, 64, 640)), (2, (2048, 2111))])
def test_transfers_of_any_length(H, lens, fp8, d):
    """The ring's transfers inside the launch: batches that a chunk does not fill, chunks of less than one."""
    import paper_2602_10940_amd as P
    wl = W.Workload("moved", 23, 1, H, d, 70, lens, "bf16")
    inp = W.make_attention_inputs(wl)
    q, k, v = dev_bf16(inp.q), [dev_bf16(x) for x in inp.k], [dev_bf16(x) for x in inp.v]
    ref_k, ref_v, kw = inp.k, inp.v, {}
    if fp8:
        packed = [[P.usp_fp8_quant(x.reshape(-1, d)) for x in t] for t in (k, v)]
        k, v = ([p[0].reshape(1, H, -1, d) for p in t] for t in packed)
        kw = {n: [p[1].reshape(1, H, -1) for p in t] for n, t in zip(("k_scales", "v_scales"), packed)}
        ref_k, ref_v = ([orc.fp8_dequant(p[0].cpu().numpy(), p[1].cpu().numpy()).reshape(1, H, -1, d) for p in t] for t in packed)
    out, lse = P.usp_ring_attn_fwd(q, k, v, softmax_scale=float(inp.softmax_scale), flags=16, **kw)
    torch.cuda.synchronize()
    ro, rl = orc.ring_attention(inp.q, ref_k, ref_v, float(inp.softmax_scale), None)
    _assert_parity(host_f64(out), host_f64(lse), ro, rl)
    if not fp8:
        plain, plse = P.usp_ring_attn_fwd(q, k, v, softmax_scale=float(inp.softmax_scale))
        torch.cuda.synchronize()
        assert torch.equal(out, plain) and torch.equal(lse, plse)
