"""How the GEMMs of a layer are distributed (tiles, K slices, one launch or two), from the planner alone: no GPU.
Figures: us measured on MI355X, with the plan asserted and with another one."""
import random

import pytest

import paper_2503_21261_amd as hot


def plan(L, O, I, **cfg):
    block = cfg.pop("block", 16)
    return hot.hot_debug_gemm_plan(hot.Config(block=block, keep=block // 2, **cfg), L, O, I)


@pytest.mark.parametrize("L,O,I,gx_bits", [
    (128, 40960, 512, 8),      # a layer pass 144, in one launch 266: g_x's 320 stages are split in eight alone
    (128, 32768, 128, 8),      # 90, 183
    (2048, 8192, 150, 4)])     # both GEMMs 26, 34
def test_long_g_x_reductions_keep_a_launch_and_their_slices(L, O, I, gx_bits):
    p = plan(L, O, I, gx_bits=gx_bits)
    assert not p["one_launch"]
    assert p["gx"] == p["gx_alone"] and p["gx"][2] > 1


@pytest.mark.parametrize("L,O,I,gx_bits", [(7872, 1664, 2757, 8), (9232, 1200, 4297, 8), (10976, 1152, 4096, 8),
                                           (512, 768, 768, 4), (12608, 3072, 768, 4), (50432, 2304, 768, 4)])
def test_short_g_x_reductions_share_g_w_s_launch(L, O, I, gx_bits):
    p = plan(L, O, I, gx_bits=gx_bits)    # the first: a backward call 149, in two launches 214
    assert p["one_launch"] and p["gx"][0] == 128 and p["gx"][2:] == (1, False)


@pytest.mark.parametrize("L,O,I,gw_bits", [(16384, 7904, 3584, 16),    # a layer pass 1193, in one launch 1262
                                           (15360, 7712, 3840, 8),     # 982, 1027
                                           (25920, 3264, 3840, 16)])   # 863, 904
def test_large_tiles_of_both_gemms_keep_their_launches(L, O, I, gw_bits):
    p = plan(L, O, I, gw_bits=gw_bits)
    assert not p["one_launch"] and p["gw"][:2] == (256, 256)


@pytest.mark.parametrize("L,O,I,gx_bits,gw_bits", [(13648, 3600, 1060, 8, 8),    # a layer pass 306, apart 368
                                                   (20816, 3840, 1113, 4, 16),   # 437, 548
                                                   (6784, 5824, 768, 4, 8),      # 181, 207
                                                   (7072, 5360, 1214, 8, 8)])    # 226, 250
def test_large_g_w_tiles_are_given_up_where_a_launch_gains_by_it(L, O, I, gx_bits, gw_bits):
    p = plan(L, O, I, gx_bits=gx_bits, gw_bits=gw_bits)
    assert p["one_launch"] and p["gw_alone"][0] == 256 and p["gw"][:2] == (128, 128)


@pytest.mark.parametrize("L,O,I,gx_bits,least", [
    (20736, 832, 2816, 4, 2),      # a layer pass 251 with g_w in two slices, unsplit 267
    (56128, 576, 912, 4, 4),       # outputs of half sectors ...
    (56128, 576, 921, 8, 4),       # ... and of broken ones, behind which g_w's loads wait
    (62640, 336, 1477, 4, 4),      # both GEMMs 143 in six slices, 190 in two
    (63904, 224, 1664, 4, 4)])     # a layer pass 330 in eight slices
def test_g_w_is_split_finer_in_front_of_many_g_x_workgroups(L, O, I, gx_bits, least):
    p = plan(L, O, I, gx_bits=gx_bits)
    assert p["one_launch"] and p["gw"][:2] == (128, 128) and p["gw"][2] >= least


@pytest.mark.parametrize("L,O,I,block,gx_bits,where,streams", [
    (12608, 3072, 768, 16, 4, "gx", True),       # whole sectors
    (2048, 4096, 11008, 64, 4, "gx_alone", False),   # a long INT4 reduction
    (11744, 256, 3079, 16, 4, "gx_alone", False),    # broken sectors: 31 us, 76 with the hint
    (608, 992, 6570, 16, 4, "gx_alone", True),       # 15.5, 16.2 without: 16 MB
    (1024, 384, 771, 16, 4, "gx_alone", False),      # 3 MB
    (16848, 1152, 2344, 16, 4, "gx", True),          # a layer pass 240, 251 without
    (5536, 576, 5434, 16, 4, "gx", False),           # 125, with it 134
    (8432, 512, 1862, 16, 4, "gx", True),
    (26592, 1376, 1332, 32, 4, "gx_alone", True),    # 124, 134 without
    (9088, 1280, 6163, 64, 4, "gx_alone", False),    # 96, with it 112
    (178432, 896, 5828, 64, 4, "gx_alone", False)])  # 1493, 1728
def test_streaming_stores_of_broken_sectors(L, O, I, block, gx_bits, where, streams):
    assert (where in plan(L, O, I, block=block, gx_bits=gx_bits)["streams"]) == streams


def test_plans_stay_within_their_limits():
    rng = random.Random(5)

    def spread(lo, hi):
        return int(lo * (hi / lo) ** rng.random())

    together = 0
    for _ in range(4000):
        block, gx_bits, gw_bits = rng.choice([16, 32, 64]), rng.choice([4, 8]), rng.choice([8, 8, 16])
        O, I, L = spread(block, 60000) // block * block, spread(1, 60000), spread(block, 250000) // block * block
        if O > 130000 or (gw_bits == 8 and L // 2 > 133144):
            continue
        p = plan(L, O, I, block=block, gx_bits=gx_bits, gw_bits=gw_bits)
        stages = -(-(L // 2 * gw_bits // 8) // 128)
        for name, rows in (("gw", O), ("gw_alone", O), ("gx", L), ("gx_alone", L)):
            bm, bn, slices, images = p[name]
            tiles = -(-rows // bm) * -(-I // bn)
            nk = stages if name[1] == "w" else -(-O * gx_bits // 8 // 128) * (2 if gx_bits == 4 else 1)
            assert (bm, bn) in ((128, 128), (128, 256), (192, 256), (256, 256))
            assert 1 <= slices <= (64 if images else 8) or name[1] == "w" and gw_bits == 16
            if slices > 1 and not images and not (name[1] == "w" and gw_bits == 16):
                assert tiles * (slices - 1) <= 1024 and (bm, bn) in ((128, 128), (256, 256))
            if slices > 1:
                assert nk // slices >= 3
        if p["one_launch"]:
            together += 1
            assert p["gw"][:2] == (128, 128) and p["gx"][0] == 128 and p["gx"][2:] == (1, False)
            assert -(-O // 128) * -(-I // 128) + -(-L // 128) * -(-I // p["gx"][1]) <= 4096
        else:
            assert p["gx"] == p["gx_alone"] and p["gw"] == p["gw_alone"]
        if gw_bits == 16:   # the bits of its sums follow from the slices: the same in every form
            assert p["gw"][2:] == p["gw_alone"][2:]
    assert together > 1000


def test_forced_distributions_make_launches_of_their_own():
    try:
        hot.hot_debug_set_gemm_mode(1)
        assert not plan(512, 768, 768)["one_launch"]
        hot.hot_debug_set_gemm_mode(0)
        hot.hot_debug_set_backward_strategy(3)
        assert not plan(512, 768, 768)["one_launch"]
    finally:
        hot.hot_debug_set_gemm_mode(0)
        hot.hot_debug_set_backward_strategy(0)
    assert plan(512, 768, 768)["one_launch"]


def test_plan_refuses_what_the_calls_refuse():
    for L, O, I in ((500, 768, 768), (512, 100, 768), (512, 768, 0)):
        with pytest.raises(hot.HotError):
            plan(L, O, I)
