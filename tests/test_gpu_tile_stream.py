"""Dead keys (ragged chunks, key masks) and shared keys in the tile stream of the matrix-core kernels: edges
of tiles, words and parts, against the fp64 oracle at the bars of the other attention tests."""
import numpy as np
import pytest
import torch

from oracle import usp_oracle as orc
from paper_2602_10940_amd import diag
from paper_2602_10940_amd import workloads as W
from tests.gpu_util import DEV, dev_bf16, host_f64
from tests.test_gpu_fp8_ring import _fp8_ring

pytestmark = pytest.mark.gpu


def _P():
    import paper_2602_10940_amd as P
    return P


def _leave_nan_in_lds(d):
    """An ordinary launch on NaN inputs: whatever the next kernel does not write in LDS is then NaN."""
    x = torch.full((1, 256, 256, d), float("nan"), device=DEV, dtype=torch.bfloat16)
    _P().usp_ring_attn_fwd(x, [x], [x])


def _parity(o, l, ro, rl):
    o, l = host_f64(o), host_f64(l)
    assert np.array_equal(np.isneginf(l), np.isneginf(rl))
    live = ~np.isneginf(rl)
    assert np.abs(o - ro).max() <= 2e-2 * max(1.0, np.abs(ro).max())
    assert np.linalg.norm(o - ro) <= 5e-3 * np.linalg.norm(ro)
    assert np.abs(l[live] - rl[live]).max() <= 1e-3


def _masks(rng, B, lens, kind):
    if kind is None:
        return None
    total = sum(lens)
    m = np.ones((B, total), np.uint8)
    for b in range(B):
        if kind == "tail":       # whole tiles of the end are dead, another number in every entry
            m[b, total - (total // 3) * (b + 1) // B - 7:] = 0
        elif kind == "holes":    # single keys, a whole tile, the first keys
            m[b, rng.integers(0, total, 9)] = 0
            m[b, 64:128] = 0
            m[b, :3] = 0
        elif kind == "all":      # one entry has no live key
            m[b, :] = 1 if b else 0
    cuts = np.cumsum(lens)[:-1]
    return [np.ascontiguousarray(x) for x in np.split(m, cuts, axis=1)]


# (B, H, Sq, lens): ragged rings in one launch (513 = one row in the last tile, 575 = one missing), one chunk
# shorter than a tile, keys shared by 2 and more work-groups, more parts than live tiles
SHAPES = [(1, 6, 300, (513, 575, 640)), (2, 2, 70, (70, 0, 69, 5)), (2, 3, 129, (700, 0, 525)), (1, 4, 40, (37,)), (2, 2, 200, (1100,)),
          (1, 1, 64, (4608,)), (1, 2, 130, (2049, 1023)), (2, 1, 257, (1024, 1024))]


@pytest.mark.parametrize("mask", [None, "tail", "holes", "all"])
@pytest.mark.parametrize("d,fp8", [(128, False), (64, False), (128, True), (64, True)])
@pytest.mark.parametrize("B,H,Sq,lens", SHAPES)
def test_dead_keys_and_parts(B, H, Sq, lens, d, fp8, mask):
    if mask == "all" and B == 1:
        pytest.skip("covered with two entries")
    P = _P()
    wl = W.Workload("stream", 17 + Sq, B, H, d, Sq, lens, "bf16")
    km = _masks(np.random.default_rng(Sq), B, lens, mask)
    if fp8:
        inp, q, k, ksc, v, vsc, kx, vx = _fp8_ring(wl)
        kw = dict(k_scales=ksc, v_scales=vsc)
    else:
        inp = W.make_attention_inputs(wl)
        q, k, v, kx, vx = dev_bf16(inp.q), [dev_bf16(x) for x in inp.k], [dev_bf16(x) for x in inp.v], inp.k, inp.v
        kw = dict()
    kw["softmax_scale"] = float(inp.softmax_scale)
    if km is not None:
        kw["key_mask"] = [torch.from_numpy(m).to(DEV) for m in km]
    ro, rl = orc.ring_attention(inp.q, kx, vx, float(inp.softmax_scale), km)
    ref = None
    for flags in (0, P.USP_ATTN_KERNEL_WIDE, P.USP_ATTN_KERNEL_SPLIT, P.USP_ATTN_FUSED_PREFETCH):
        _leave_nan_in_lds(d)
        desc = P.make_attn_desc(q, k, q, kw["softmax_scale"], flags)
        ws = torch.full((P.usp_ring_attn_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device=DEV)
        o, l = P.usp_ring_attn_fwd(q, k, v, flags=flags, workspace=ws, **kw)
        torch.cuda.synchronize()
        _parity(o, l, ro, rl)
        if flags == 0:
            ref = o, l
        elif flags == P.USP_ATTN_FUSED_PREFETCH:     # the transfers inside the launch change no bit
            assert torch.equal(o, ref[0]) and torch.equal(l, ref[1])


# short chunks travel side by side in up to eight groups of the copy work-groups: fewer later chunks than
# groups, as many, more (two for some groups), the most that one launch takes
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lens", [(64, 64), (64, 128, 64, 64), (64,) * 9, (128, 0, 64) + (64,) * 9, (64,) * 16])
def test_short_chunks_travel_side_by_side(lens, d, fp8):
    P = _P()
    wl = W.Workload("groups", 40 + len(lens), 2, 3, d, 200, lens, "bf16")
    if fp8:
        inp, q, k, ksc, v, vsc, kx, vx = _fp8_ring(wl)
        kw = dict(k_scales=ksc, v_scales=vsc)
    else:
        inp = W.make_attention_inputs(wl)
        q, k, v, kx, vx = dev_bf16(inp.q), [dev_bf16(x) for x in inp.k], [dev_bf16(x) for x in inp.v], inp.k, inp.v
        kw = dict()
    kw["softmax_scale"] = float(inp.softmax_scale)
    ro, rl = orc.ring_attention(inp.q, kx, vx, kw["softmax_scale"])
    plain = P.usp_ring_attn_fwd(q, k, v, **kw)
    desc = P.make_attn_desc(q, k, q, kw["softmax_scale"], P.USP_ATTN_FUSED_PREFETCH)
    ws = torch.empty((P.usp_ring_attn_workspace_bytes(desc),), dtype=torch.uint8, device=DEV)
    for _ in range(3):
        ws.fill_(0xFF)
        o, l = P.usp_ring_attn_fwd(q, k, v, flags=P.USP_ATTN_FUSED_PREFETCH, workspace=ws, **kw)
        torch.cuda.synchronize()
        _parity(o, l, ro, rl)
        assert torch.equal(o, plain[0]) and torch.equal(l, plain[1])


@pytest.mark.parametrize("d,Sq,lens", [(128, 1800, (64, 128, 64)), (128, 1700, (600, 500)), (64, 1800, (128, 64, 192))])
def test_short_chunks_under_more_than_one_round_of_query_blocks(d, Sq, lens):
    """40 heads with seven or eight 256-query blocks each: the plain call takes these rings as one launch."""
    inp = W.make_attention_inputs(W.Workload("rounds", 3 + Sq, 1, 40, d, Sq, lens, "bf16"))
    ro, rl = orc.ring_attention(inp.q, inp.k, inp.v, float(inp.softmax_scale))
    o, l = _P().usp_ring_attn_fwd(dev_bf16(inp.q), [dev_bf16(x) for x in inp.k], [dev_bf16(x) for x in inp.v],
                                  softmax_scale=float(inp.softmax_scale))
    torch.cuda.synchronize()
    _parity(o, l, ro, rl)


@pytest.mark.parametrize("d,Sc,masked,flags", [(128, 64, True, 4), (128, 64, True, 8), (128, 100, False, 4), (128, 100, False, 8),
                                               (64, 100, True, 0), (72, 100, True, 0), (72, 64, False, 0)])
def test_token_strides_at_the_end_of_32_bits(d, Sc, masked, flags):
    """Keys 64 MB apart: a tile's 64 steps are 2^32 bytes (d = 72: past what the general kernel reaches with 32 bits)."""
    P = _P()
    step = 1 << 25                                    # elements
    store = torch.empty(((Sc - 1) * step + 2048,), dtype=torch.bfloat16, device=DEV)
    k, v = (store.as_strided((1, 2, Sc, d), (step, 512, step, 1), off) for off in (0, 1024))
    g = torch.Generator(device=DEV)
    g.manual_seed(d + Sc)
    for t in (k, v):
        t.copy_(torch.randn((1, 2, Sc, d), generator=g, device=DEV))
    q = torch.randn((1, 2, 50, d), generator=g, device=DEV).bfloat16()
    keep = torch.ones((1, Sc), dtype=torch.uint8, device=DEV)
    if masked:
        keep[0, 3], keep[0, 60:63] = 0, 0
    o, l = P.usp_ring_attn_fwd(q, [k], [v], key_mask=[keep] if masked else None, flags=flags)
    z = torch.matmul(q.float(), k.float().transpose(2, 3).contiguous()) * d ** -0.5
    z = z.masked_fill(keep[0] == 0, float("-inf"))
    _parity(o, l, host_f64(torch.softmax(z, -1) @ v.float()), host_f64(torch.logsumexp(z, -1)))


def test_the_mixed_form_of_a_ring_is_a_launch_per_chunk():
    P = _P()
    inp = W.make_attention_inputs(W.Workload("mixed", 8, 1, 40, 128, 1800, (64, 128, 64), "bf16"))
    q, k, v = dev_bf16(inp.q), [dev_bf16(x) for x in inp.k], [dev_bf16(x) for x in inp.v]
    o, l = P.usp_ring_attn_fwd(q, k, v, flags=P.USP_ATTN_KERNEL_MIXED)
    o2, l2 = P.usp_ring_attn_fwd(q, k, v, flags=P.USP_ATTN_KERNEL_MIXED | P.USP_ATTN_STEPWISE)
    torch.cuda.synchronize()
    assert torch.equal(o, o2) and torch.equal(l, l2)


def test_parts_need_no_more_workspace_than_there_is():
    """A workspace that holds a launch per chunk but not the parts is enough; one byte less is refused."""
    P = _P()
    inp = W.make_attention_inputs(W.Workload("least", 5, 1, 1, 128, 128, (4608,), "bf16"))
    q, k, v = dev_bf16(inp.q), [dev_bf16(x) for x in inp.k], [dev_bf16(x) for x in inp.v]
    least = 72 * 1024 + 256                          # 1 KB per tile of the head, one count
    assert P.usp_ring_attn_workspace_bytes(P.make_attn_desc(q, k, q)) > least
    ro, rl = orc.ring_attention(inp.q, inp.k, inp.v, float(inp.softmax_scale))
    o, l = P.usp_ring_attn_fwd(q, k, v, softmax_scale=float(inp.softmax_scale),
                               workspace=torch.empty((least,), dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    _parity(o, l, ro, rl)
    with pytest.raises(P.UspError):
        P.usp_ring_attn_fwd(q, k, v, workspace=torch.empty((least - 1,), dtype=torch.uint8, device=DEV))


@pytest.mark.parametrize("split", [False, True, None])
@pytest.mark.parametrize("n", [1, 2])
def test_more_dead_tiles_than_words(n, split):
    """250 007 keys, ragged and masked: beyond the words a work-group keeps in LDS.  None: the plain call, which
    shares the keys of the one chunk between work-groups.  Reference in fp32."""
    P = _P()
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    total, Sq = 250007, 96
    q, k, v = (torch.randn((1, 1, s, 128), generator=g, device=DEV).bfloat16() for s in (Sq, total, total))
    keep = torch.ones((1, total), dtype=torch.uint8, device=DEV)
    keep[:, 1000:1500] = 0
    keep[:, total - 70000:] = 0
    lens = (total,) if n == 1 else (130001, total - 130001)
    flags = 0 if split is None else P.USP_ATTN_KERNEL_SPLIT if split else P.USP_ATTN_KERNEL_WIDE
    ks, vs = [x.contiguous() for x in k.split(lens, 2)], [x.contiguous() for x in v.split(lens, 2)]
    route = diag.usp_diag_attn_route(P.make_attn_desc(q, ks, q, flags=flags), masked=True)
    assert not route.one_launch and (route.parts > 1) == (split is None and n == 1)
    o, l = P.usp_ring_attn_fwd(q, ks, vs, key_mask=[x.contiguous() for x in keep.split(lens, 1)], flags=flags)
    s = (q[0, 0].float() @ k[0, 0].float().T) * 128 ** -0.5
    s = s.masked_fill(keep[0] == 0, float("-inf"))
    ro, rl = torch.softmax(s, -1) @ v[0, 0].float(), torch.logsumexp(s, -1)
    _parity(o, l, host_f64(ro[None, None]), host_f64(rl[None, None]))


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("flags", [0, 4, 8])
@pytest.mark.parametrize("Sc,n", [(37, 1), (97, 1), (1000, 1), (545, 2)])
def test_nothing_behind_a_ragged_chunk_is_read(d, flags, Sc, n):
    """The rows behind each head's last key are NaN: they load as zeros, in the lower and the upper half of a tile."""
    P = _P()
    B, H, Sq = 2, 2, 140
    inp = W.make_attention_inputs(W.Workload("behind", 60 + Sc, B, H, d, Sq, (Sc,) * n, "bf16"))

    def view(x):
        store = torch.full((B, H, Sc + 64, d), float("nan"), dtype=torch.bfloat16, device=DEV)
        store[:, :, :Sc] = dev_bf16(x)
        return store[:, :, :Sc]
    o, l = P.usp_ring_attn_fwd(dev_bf16(inp.q), [view(k) for k in inp.k], [view(v) for v in inp.v],
                               softmax_scale=float(inp.softmax_scale), flags=flags)
    torch.cuda.synchronize()
    ro, rl = orc.ring_attention(inp.q, inp.k, inp.v, float(inp.softmax_scale))
    _parity(o, l, ro, rl)
