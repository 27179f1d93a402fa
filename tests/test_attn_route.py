"""Which launches usp_ring_attn_fwd chooses (usp_diag_attn_route: host code, no GPU)."""
import ctypes

import pytest

from paper_2602_10940_amd import binding as b
from paper_2602_10940_amd import diag


def _desc(B, H, d, Sq, lens, fp8=False, flags=0, f32=False):
    x = b.AttnDesc()
    x._lens = (ctypes.c_int32 * len(lens))(*lens)
    x.B, x.H, x.d, x.Sq, x.n_chunks, x.flags = B, H, d, Sq, len(lens), flags
    x.chunk_len = ctypes.cast(x._lens, ctypes.POINTER(ctypes.c_int32))
    x.qo_dtype = b.USP_F32 if f32 else b.USP_BF16
    x.kv_dtype = b.USP_FP8_E4M3FN if fp8 else x.qo_dtype
    for i, s in enumerate((H * Sq * d, Sq * d, d)):
        x.q_stride[i] = x.o_stride[i] = s
    return x


def _route(*a, masked=False, **kw):
    return diag.usp_diag_attn_route(_desc(*a, **kw), masked)


# rings whose chunks arrive later than few tiles of keys take: sharing the keys was slower there by 13 to 43 %
SHORT = [(2, 12, 128, 150, (320,) * 8, True), (2, 11, 128, 576, (576,) * 8, True), (2, 18, 128, 70, (395,) * 3, True),
         (1, 7, 64, 102, (384,) * 3, False), (1, 16, 64, 82, (192,) * 6, False)]


@pytest.mark.parametrize("B,H,d,Sq,lens,fp8", SHORT)
def test_short_chunks_that_arrive_late_keep_their_keys_together(B, H, d, Sq, lens, fp8):
    assert _route(B, H, d, Sq, lens, fp8=fp8, flags=b.USP_ATTN_FUSED_PREFETCH)[::2] == (True, 1)


@pytest.mark.parametrize("fp8", [False, True])
def test_long_chunks_under_few_queries_share_their_keys(fp8):
    for lens in ((2816,) * 6, (2816,)):
        one, _, parts = _route(1, 2, 128, 108, lens, fp8=fp8)
        assert one == (len(lens) > 1) and parts >= 8


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lens", [(64,) * 8, (128, 640), (384,) * 8, (513, 575, 640), (2816,) * 4])
def test_transfers_inside_the_launch_do_not_change_the_form(d, lens):
    for H, Sq in ((1, 64), (2, 300), (5, 640), (12, 100)):
        assert _route(1, H, d, Sq, lens) == _route(1, H, d, Sq, lens, flags=b.USP_ATTN_FUSED_PREFETCH)


# B, H, d, Sq, keys, parts: launches that the first rule gives parts (whose number stays: fewer would be further from 64 bits), those that gain by
# the times of today (the fastest of 1, 2, 3, 4, 6 and 8 or within 2 % of it), and those that gain by neither
SHARED = [(1, 5, 64, 112, 3648, (15,)), (1, 1, 64, 936, 985, (16,)), (2, 2, 128, 241, 1568, (13,)), (1, 3, 128, 4608, 4608, (2,)),
          (2, 2, 64, 3861, 3456, (2,)), (1, 2, 128, 1399, 1024, (3, 4)), (1, 13, 64, 187, 960, (3, 4)), (1, 12, 64, 416, 576, (1,)),
          (2, 13, 64, 2049, 640, (1,)), (2, 2, 128, 1937, 384, (1,)), (2, 14, 128, 737, 960, (1,))]


@pytest.mark.parametrize("B,H,d,Sq,keys,parts", SHARED)
def test_parts_of_one_chunk(B, H, d, Sq, keys, parts):
    got = _route(B, H, d, Sq, (keys,)).parts
    assert got in parts
    need = b.usp_ring_attn_workspace_bytes(_desc(B, H, d, Sq, (keys,)))
    assert got == 1 or need >= 4 * got * B * H * Sq * (d + 2)


# B, H, Sq, keys, masked: FP8, d = 64.  Dead keys (a mask, a ragged end) leave one work-group to a CU, whole unmasked tiles two
CROWDED = [(1, 11, 1500, 4500, False), (1, 9, 2048, 4600, False), (1, 13, 1500, 4500, False), (1, 17, 1000, 4608, True), (1, 17, 1000, 4600, False),
           (1, 17, 1000, 4600, True), (1, 8, 2100, 3500, False), (2, 5, 2048, 4608, True), (1, 30, 1024, 16384, True)]


@pytest.mark.parametrize("B,H,Sq,keys,masked", CROWDED)
def test_parts_of_a_form_with_one_work_group_to_a_cu_take_one_round(B, H, Sq, keys, masked):
    """More than 120 work-groups undivided: two parts would be a second round of work-groups."""
    assert 120 < 8 * -(-B * H * -(-Sq // 128) // 8) <= 240
    assert _route(B, H, 64, Sq, (keys,), fp8=True, masked=masked).parts == 1


def test_a_mask_takes_parts_only_from_the_form_that_it_changes():
    assert _route(1, 17, 64, 1000, (4608,), fp8=True).parts > 1
    for B, H, d, Sq, keys, parts in SHARED:      # bf16: the same with a mask
        assert _route(B, H, d, Sq, (keys,), masked=True) == _route(B, H, d, Sq, (keys,))
    for H, Sq, keys in ((2, 300, 4096), (6, 1500, 3000), (1, 64, 960)):      # FP8, few query blocks: parts within one round, mask or not
        for k in (keys // 64 * 64, keys // 64 * 64 - 1):
            for masked in (False, True):
                parts = _route(1, H, 64, Sq, (k,), fp8=True, masked=masked).parts
                assert parts > 1 and (parts * 8 * -(-H * -(-Sq // 128) // 8) <= 240 or not (masked or k % 64))
        whole = (keys // 64 * 64,)               # the workspace has room for either
        most = max(_route(1, H, 64, Sq, whole, fp8=True, masked=m).parts for m in (False, True))
        assert b.usp_ring_attn_workspace_bytes(_desc(1, H, 64, Sq, whole, fp8=True)) >= 4 * H * Sq * 66 * most


def test_parts_never_outnumber_what_a_second_launch_takes():
    for d in (64, 128):
        for heads in (1, 2, 7, 24, 60):
            for Sq in (1, 129, 500, 4608):
                for keys in (1, 64, 65, 513, 4097, 70000):
                    blocks = 8 * -(-heads * -(-Sq // 128) // 8)
                    for lens, most in (((keys,), 480 if d == 64 else 240), ((64 * -(-keys // 64),) * 2, 240)):
                        parts = _route(1, heads, d, Sq, lens).parts
                        assert 1 <= parts <= 16 and (parts == 1 or (parts * blocks <= most and parts <= sum(-(-n // 64) for n in lens)))


# us of a launch per chunk, one launch of 256-query work-groups, one key-split launch (all chunks at hand)
MEASURED = [(2, 24, 128, 4608, 2, 1536, 370, 331, 363), (1, 22, 128, 3112, 2, 128, 57, 32, 39), (1, 24, 128, 2816, 4, 1024, 245, 208, 184),
            (1, 20, 128, 3500, 3, 2048, 302, 302, 261), (2, 13, 128, 2384, 6, 256, 214, 92, 64), (2, 21, 128, 1865, 8, 1216, 563, 470, 410),
            (2, 18, 128, 3629, 2, 3008, 430, 456, 432)]
# d = 64, two key-split work-groups to a CU.  us of a launch per chunk (any form, 256-query, key-split), one launch of 256-query work-groups, one
# key-split launch, and these two with the transfers inside
MEASURED_64 = [(2, 22, 4416, 2, 128, (66.2, 66.5, 57.1), (36.7, 34.1), (42.8, 44.9)), (2, 19, 3621, 2, 128, (49.7, 49.5, 43.3), (27.1, 24.4), (32.3, 35.3)),
               (2, 15, 2149, 6, 384, (86.7, 142.1, 86.1), (82.3, 44.1), (88.9, 66.6)), (2, 22, 1725, 6, 3328, (498.6, 701.5, 494.5), (633.2, 445.0), (634.8, 478.9)),
               (2, 14, 4544, 2, 960, (79.8, 90.6, 80.1), (71.5, 68.6), (83.6, 74.0)), (1, 24, 4608, 2, 2304, (155.4, 171.1, 155.6), (154.6, 144.9), (155.6, 146.5)),
               (1, 17, 4300, 8, 512, (173.4, 230.4, 173.3), (137.9, 100.4), (146.2, 119.7)), (1, 17, 5000, 2, 128, (29.1, 32.8, 29.1), (18.9, 16.6), (22.8, 26.1)),
               (1, 17, 5000, 2, 192, (31.5, 37.1, 31.5), (22.5, 19.2), (24.9, 23.3)), (2, 24, 3900, 8, 832, (424.0, 498.8, 424.9), (335.8, 316.3), (377.4, 326.9)),
               (1, 300, 100, 2, 128, (18.0, 26.3, 18.0), (18.3, 12.0), (31.4, 25.5)), (1, 24, 4096, 12, 128, (205.0, 233.7, 204.7), (60.2, 49.3), (74.4, 68.6)),
               (1, 20, 4608, 2, 11264, (525.3, 733.9, 522.5), (721.6, 511.9), (722.7, 515.3)), (1, 17, 4096, 2, 320, (34.3, 42.9, 34.7), (30.3, 24.1), (32.8, 27.5)),
               (2, 17, 2921, 8, 512, (249.9, 248.9, 221.6), (139.7, 130.5), (150.0, 160.8))]


@pytest.mark.parametrize("B,H,d,Sq,n,chunk,stepwise,wide,split", MEASURED)
def test_more_than_one_round_of_query_blocks_runs_the_form_that_was_judged(B, H, d, Sq, n, chunk, stepwise, wide, split):
    r = _route(B, H, d, Sq, (chunk,) * n)
    took = stepwise if not r.one_launch else split if r.split else wide
    assert took <= 1.05 * min(stepwise, wide, split)
    # the transfers inside the launch: the same form
    pre = _route(B, H, d, Sq, (chunk,) * n, flags=b.USP_ATTN_FUSED_PREFETCH)
    assert pre.one_launch and (not r.one_launch or pre.split == r.split)
    # a forced form is judged by what it costs itself
    for flag, us in ((b.USP_ATTN_KERNEL_WIDE, wide), (b.USP_ATTN_KERNEL_SPLIT, split)):
        f = _route(B, H, d, Sq, (chunk,) * n, flags=flag)
        assert (us if f.one_launch else stepwise) <= 1.05 * min(us, stepwise)
        assert not f.one_launch or f.split == (flag == b.USP_ATTN_KERNEL_SPLIT)


@pytest.mark.parametrize("B,H,Sq,n,chunk,stepwise,at_hand,inside", MEASURED_64)
def test_d64_rings_above_one_round_run_the_faster_form(B, H, Sq, n, chunk, stepwise, at_hand, inside):
    """One form for both ways a ring's chunks come: the faster with the chunks at hand, unless that is the slower one with the transfers inside."""
    lens, pre = (chunk,) * n, b.USP_ATTN_FUSED_PREFETCH
    r, p = _route(B, H, 64, Sq, lens), _route(B, H, 64, Sq, lens, flags=pre)
    assert B * H * -(-Sq // 256) > 256 and r.one_launch and p.one_launch and r.split == p.split
    assert inside[r.split] <= 1.05 * min(inside)
    assert at_hand[r.split] <= 1.05 * min(at_hand) or inside[not r.split] > inside[r.split]
    for split, flag in ((False, b.USP_ATTN_KERNEL_WIDE), (True, b.USP_ATTN_KERNEL_SPLIT)):      # a forced form, against a launch per chunk in that form
        f = _route(B, H, 64, Sq, lens, flags=flag)
        assert f.one_launch and f.split == split and at_hand[split] <= 1.05 * stepwise[1 + split]
    assert min(at_hand) <= min(stepwise)


@pytest.mark.parametrize("B,H,Sq,lens,split", [(1, 17, 5000, (128, 64), False), (1, 17, 5000, (192, 192), True), (1, 17, 5000, (320, 321), True),
                                               (1, 300, 100, (64, 64), True), (1, 24, 4608, (2304, 2304), True), (1, 24, 4608, (2303, 2302), True)])
def test_d64_rings_from_fp8_are_not_taken_for_two_work_groups_to_a_cu(B, H, Sq, lens, split):
    """FP8 chunks keep one key-split work-group to a CU; dead keys change nothing about bf16 ones."""
    pre = b.USP_ATTN_FUSED_PREFETCH
    assert [_route(B, H, 64, Sq, lens, flags=pre, masked=m).split for m in (False, True)] == [split, split]
    tiles, blocks, halves = sum(-(-n // 64) for n in lens), B * H * -(-Sq // 256), B * H * -(-Sq // 128)
    wide = -(-blocks // 256) * (8.0 + 1.13 * tiles)
    assert _route(B, H, 64, Sq, lens, fp8=True, flags=pre).split == (-(-halves // 256) * (7.1 + 0.47 * tiles) + 0.16 * tiles * halves / 256 < wide)


@pytest.mark.parametrize("H,n,fp8", [(12, 3, False), (12, 8, False), (8, 8, False), (20, 3, False), (12, 2, True)])
def test_the_route_does_not_depend_on_the_scratch_of_another_entry_point(H, n, fp8):
    """Ragged rings whose one launch needs more workspace than the library's own scratch holds: the caller
    brings it, so they take the one launch, as the plain call does (whose bits they promise)."""
    lens, pre = (2215,) * n, b.USP_ATTN_FUSED_PREFETCH
    plain, inside = _route(1, H, 128, 2215, lens, fp8=fp8), _route(1, H, 128, 2215, lens, fp8=fp8, flags=pre)
    assert inside.one_launch and (fp8 or plain == inside)
    full = b.usp_ring_attn_workspace_bytes(_desc(1, H, 128, 2215, lens, fp8, pre))
    assert full > b.usp_ring_attn_workspace_bytes(_desc(1, H, 128, 2215, lens, fp8, pre | b.USP_ATTN_STEPWISE))
    if full <= b.USP_NOALLOC_SCRATCH_BYTES:
        return
    # what fits the scratch with a launch per chunk is not refused there for want of workspace
    least = b.usp_ring_attn_workspace_bytes(_desc(1, H, 128, 2215, lens, fp8, pre | b.USP_ATTN_STEPWISE))
    st = b.load_library().usp_ring_attn_fwd_noalloc(ctypes.byref(_desc(1, H, 128, 2215, lens, fp8, pre)), *[None] * 9)
    assert (st == b.USP_ERR_WORKSPACE) == (least > b.USP_NOALLOC_SCRATCH_BYTES) and st != b.USP_OK


@pytest.mark.parametrize("lens,fp8,pre,masked", [((64, 128, 64), False, 0, False), ((513, 640), False, 0, False),
                                                 ((513, 640), False, b.USP_ATTN_FUSED_PREFETCH, False),
                                                 ((513, 640), True, 0, False), ((512, 640), False, 0, True)])
def test_the_mixed_form_is_honoured_by_a_launch_per_chunk(lens, fp8, pre, masked):
    H, Sq = (40, 1800) if not pre and not fp8 and lens[0] == 64 else (6, 300)     # more than one round of query blocks, or ragged
    assert _route(1, H, 128, Sq, lens, fp8=fp8, flags=pre, masked=masked).one_launch
    assert not _route(1, H, 128, Sq, lens, fp8=fp8, flags=pre | b.USP_ATTN_KERNEL_MIXED, masked=masked).one_launch


def test_the_mixed_form_is_ignored_where_it_always_was():
    assert _route(1, 6, 128, 300, (512, 640), flags=b.USP_ATTN_KERNEL_MIXED).one_launch
    assert _route(1, 40, 128, 1800, (64, 128), flags=b.USP_ATTN_KERNEL_MIXED | b.USP_ATTN_FUSED_PREFETCH).one_launch
    assert _route(1, 6, 64, 300, (513, 640), flags=b.USP_ATTN_KERNEL_MIXED).one_launch      # (d = 64 has no such form)


@pytest.mark.parametrize("B,H,d,Sq,lens", [(1, 64, 128, 1025, (64, 64)), (1, 64, 128, 1025, (2048, 2048)), (2, 129, 128, 20, (65, 1, 0, 130)),
                                           (1, 64, 64, 1025, (1408, 1407)), (1, 64, 64, 1025, (256,) * 8), (1, 24, 128, 4096, (4096, 4096))])
def test_fp8_rings_at_hand_above_one_round_of_query_blocks_are_a_launch_per_chunk(B, H, d, Sq, lens):
    assert not _route(B, H, d, Sq, lens, fp8=True).one_launch
    assert b.usp_ring_attn_workspace_bytes(_desc(B, H, d, Sq, lens, True)) == \
        b.usp_ring_attn_workspace_bytes(_desc(B, H, d, Sq, lens, True, b.USP_ATTN_STEPWISE))
    assert _route(B, H, d, Sq, lens, fp8=True, flags=b.USP_ATTN_FUSED_PREFETCH).one_launch
    assert _route(1, 2, d, 75, lens, fp8=True).one_launch                                # within one round


@pytest.mark.parametrize("lens", [(38, 38), (219, 1, 0, 63, 65), (33,) * 16, (288,) * 4, (300, 318)])
@pytest.mark.parametrize("H,Sq", [(2, 75), (40, 1800)])
@pytest.mark.parametrize("flags", [0, b.USP_ATTN_FUSED_PREFETCH, b.USP_ATTN_DOUBLE_BUFFER])
def test_short_ragged_bf16_rings_are_a_launch_per_chunk(lens, H, Sq, flags):
    for d in (64, 128):
        assert not _route(1, H, d, Sq, lens, flags=flags).one_launch
        assert b.usp_ring_attn_workspace_bytes(_desc(1, H, d, Sq, lens, flags=flags)) == \
            b.usp_ring_attn_workspace_bytes(_desc(1, H, d, Sq, lens, flags=flags | b.USP_ATTN_STEPWISE))
    if flags != b.USP_ATTN_DOUBLE_BUFFER:
        assert _route(1, 2, 128, 75, (320, 321), flags=flags).one_launch and _route(1, 2, 128, 75, (64, 64), flags=flags).one_launch


def test_copy_work_groups_of_a_mixed_launch_find_their_cus_free():
    for blocks in range(1, 2600):
        plain, g = diag.usp_diag_mixed_grid(blocks), diag.usp_diag_mixed_grid(blocks, copies=True)
        rem, per = blocks % 256, -(-blocks // 8)
        assert (plain.wgs > 0) == (g.wgs > 0) == (0 < rem <= 128)
        if not g.wgs:
            continue
        last = -(-rem // 8)                                        # the last round's blocks alone
        for x in (plain, g):
            assert x.wgs == 8 * (per + x.halves) and last <= x.halves <= max(last, (per + 1) // 2)
            assert x.halves == last or x.wgs <= 256 * -(-8 * per // 256)   # no round more
        assert plain.copy_wgs == 0 and g.halves <= plain.halves
        if g.halves > last:
            assert g.copy_wgs == 64 and g.wgs + g.copy_wgs <= 256 * -(-8 * per // 256)
        else:
            assert g.wgs == 8 * (per + last)


@pytest.mark.parametrize("blocks,wgs,copies_wgs,copy_wgs", [(264, 400, 400, 64), (343, 512, 448, 64), (520, 768, 704, 64), (384, 512, 512, 64)])
def test_mixed_launches_by_number(blocks, wgs, copies_wgs, copy_wgs):
    assert diag.usp_diag_mixed_grid(blocks).wgs == wgs and diag.usp_diag_mixed_grid(blocks, copies=True)[::2] == (copies_wgs, copy_wgs)
    assert diag.usp_diag_mixed_grid(blocks, forced=True).halves == -(-((blocks + 1) // 2) // 8)


# B, H, d, Sq, keys, fp32, from FP8: the number of work-groups that share the keys of a query block in the general kernel
GENERAL = [(1, 8, 32, 102, 1549, True, False, 8), (1, 8, 128, 102, 1549, True, False, 8), (1, 4, 64, 512, 512, True, False, 4),
           (1, 4, 32, 512, 512, True, False, 1), (1, 16, 40, 153, 1793, False, False, 8), (1, 16, 160, 153, 1793, False, False, 4),
           (1, 16, 112, 153, 1793, False, True, 4), (2, 16, 72, 1024, 1024, False, False, 1), (1, 2, 64, 128, 256, True, False, 1)]


@pytest.mark.parametrize("B,H,d,Sq,keys,f32,fp8,parts", GENERAL)
def test_general_calls_over_one_chunk_under_few_queries_share_their_keys(B, H, d, Sq, keys, f32, fp8, parts):
    assert _route(B, H, d, Sq, (keys,), fp8=fp8, f32=f32) == (False, False, parts)
    # several chunks are merged one after another and keep their keys together, also where one alone holds any
    for lens in ((keys // 2, keys - keys // 2), (keys, 0), (0, keys)):
        assert _route(B, H, d, Sq, lens, fp8=fp8, f32=f32).parts == 1


@pytest.mark.parametrize("f32", [True, False])
@pytest.mark.parametrize("d", [8, 40, 72, 96, 128, 136, 160, 168, 256])
def test_the_shares_of_a_general_call(d, f32):
    if not f32 and d == 128:
        return                                                                  # (a matrix-core kernel's)
    for heads in (1, 3, 8, 24, 60, 255, 256):
        for Sq in (1, 17, 100, 513, 2048):
            for keys in (1, 64, 192, 193, 256, 257, 1024, 4097, 70000):
                parts = _route(1, heads, d, Sq, (keys,), f32=f32).parts
                need = b.usp_ring_attn_workspace_bytes(_desc(1, heads, d, Sq, (keys,), f32=f32))
                if heads * -(-Sq // 64) >= 256 or d > 160 or (f32 and d > 128) or keys <= 192:
                    assert parts == 1
                assert parts in (1, 2, 4, 8) and 2 * parts <= max(2, -(-keys // 64))      # two tiles each at least
                assert parts == 1 or parts * heads * -(-Sq // (16 if f32 else 32)) <= 768
                # fp32 O~ and (m, l) of every share, and nothing where the keys stay together
                rows = heads * Sq
                assert need == (0 if parts == 1 else sum(-(-4 * n * parts * rows // 256) * 256 for n in (d, 2)))


@pytest.mark.parametrize("kind,most", [(0, 16), (1, 8), (2, 8)])
def test_more_parts_than_the_second_launch_holds_are_refused_in_front_of_the_first(kind, most):
    for parts in (most + 1, 2 * most, 1 << 20):
        with pytest.raises(b.UspError, match="at most %d work-groups \\(got %d\\)" % (most, parts)) as e:
            diag.usp_diag_too_many_parts(kind, parts)
        assert e.value.status == b.USP_ERR_INVALID_ARG
