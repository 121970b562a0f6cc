"""Which launches the sizes choose, on both sides of the lines that were measured
(no GPU needed: the choice is a host computation)."""
import pytest

from paper_2511_13198_amd import pdyattn as P


def shapes(lengths, hq, hkv, d, causal):
    return P.launch_shapes(sum(lengths), len(lengths), max(lengths), hq, hkv, d, causal)


@pytest.mark.parametrize("lengths,hq,hkv,d,causal,expect", [
    # unsplit, 256-key tiles on part of the chip: two query groups only while
    # their 128-key workgroups fit one round and have a few steps
    ([512] * 64, 1, 1, 128, True, (8, 2, 1)),
    ([1024] * 32, 1, 1, 64, False, (8, 2, 1)),
    ([1024] * 33, 1, 1, 64, False, (8, 1, 1)),
    ([1024] * 60, 1, 1, 128, True, (8, 1, 1)),
    ([512] * 100, 1, 1, 128, False, (8, 1, 1)),
    ([2048] * 30, 1, 1, 128, False, (8, 1, 1)),
    ([192] * 8, 2, 2, 128, True, (8, 1, 1)),
    # two parts: two groups without parts
    ([2048] * 16, 1, 1, 64, True, (8, 2, 1)),
    ([4096] * 15, 1, 1, 128, False, (8, 2, 1)),
    # four parts: by the share of time that their partial results take
    ([2048] * 4, 2, 2, 128, True, (8, 2, 2)),
    ([2048] * 4, 8, 2, 128, True, (8, 1, 4)),
    ([2048] * 4, 2, 2, 64, True, (8, 2, 2)),
    ([2048] * 3, 4, 2, 64, True, (8, 1, 4)),
    ([103, 52] * 5, 32, 8, 128, True, (8, 2, 2)),
    ([103, 52] * 5, 32, 8, 64, True, (8, 2, 2)),
    ([828] * 4 + [207] * 38, 9, 3, 128, True, (8, 2, 2)),
    ([4096] * 8, 1, 1, 128, True, (8, 1, 4)),
    ([16384] * 3, 1, 1, 64, True, (8, 1, 4)),
])
def test_packed_dkdv_groups(lengths, hq, hkv, d, causal, expect):
    assert shapes(lengths, hq, hkv, d, causal)["bwd_dkdv_kernel"] == expect


@pytest.mark.parametrize("lengths,hq,fwd,dq", [
    # few heads: 4-wave query tiles only in unsplit launches up to 448 workgroups
    ([4096] * 8, 4, (8, 1, 1), (8, 1, 1)),       # 512
    ([4096] * 7, 4, (4, 1, 1), (8, 1, 2)),       # 448; dQ in parts
    ([8192] * 5, 4, (8, 1, 1), (8, 1, 1)),       # 640
    ([7697, 6000, 5554, 4800], 4, (8, 1, 2), (8, 1, 2)),
    # six heads or more: up to 767
    ([4096] * 7, 6, (4, 1, 1), (4, 1, 1)),       # 672
    ([4096] * 6, 8, (8, 1, 1), (8, 1, 1)),       # 768
    # a single sequence's line stays
    ([16384], 8, (4, 1, 1), (4, 1, 1)),
])
def test_d64_four_wave_query_tiles(lengths, hq, fwd, dq):
    got = shapes(lengths, hq, hq, 64, True)
    assert (got["fwd_kernel"], got["bwd_dq_kernel"]) == (fwd, dq)


@pytest.mark.parametrize("T,hq,hkv,d,causal,fwd,dq,dkdv", [
    # split launches: half of the parts and two groups where that saves enough
    (8192, 4, 4, 128, True, (8, 2, 2), (8, 2, 2), (8, 2, 2)),
    (16128, 4, 4, 128, True, (8, 1, 4), (8, 2, 2), (8, 2, 2)),
    (16384, 4, 4, 128, True, (8, 1, 2), (8, 2, 1), (8, 2, 1)),
    (13433, 3, 3, 64, True, (8, 1, 4), (8, 1, 4), (8, 1, 4)),
    (8192, 8, 8, 64, True, (8, 2, 1), (8, 2, 1), (8, 2, 1)),
    (8853, 8, 8, 64, True, (8, 1, 2), (8, 1, 2), (8, 2, 1)),
    (8192, 8, 8, 64, False, (8, 1, 2), (8, 1, 2), (8, 1, 2)),
    # groups need 256 keys
    (255, 4, 4, 64, True, (4, 1, 1), (4, 1, 1), (8, 2, 1)),
    (256, 4, 4, 64, True, (8, 4, 1), (8, 4, 1), (8, 2, 1)),
    # more than a round: not at d = 64 without a mask, nor (much more) for a
    # causal forward
    (24701, 8, 4, 64, False, (8, 1, 1), (8, 1, 1), (8, 1, 2)),
    (2901, 32, 16, 128, True, (8, 1, 1), (8, 2, 1), (8, 2, 2)),
    # 4-wave query tiles at d = 64: dQ with few heads up to two rounds
    (38243, 4, 4, 64, True, (4, 1, 1), (8, 1, 1), (8, 1, 1)),
    (17045, 8, 8, 64, True, (4, 1, 1), (4, 1, 1), (8, 1, 1)),
    # 4-wave dQ up to a round (168 and 256 workgroups): four groups; beyond: none
    (1789, 12, 4, 64, True, (8, 4, 1), (8, 4, 1), (8, 2, 8)),
    (2048, 16, 16, 128, True, (8, 4, 1), (8, 4, 1), (8, 2, 1)),
    (2048, 17, 17, 128, True, (4, 1, 1), (4, 1, 1), (8, 2, 1)),
])
def test_single_sequences(T, hq, hkv, d, causal, fwd, dq, dkdv):
    got = shapes([T], hq, hkv, d, causal)
    assert (got["fwd_kernel"], got["bwd_dq_kernel"], got["bwd_dkdv_kernel"]) == (fwd, dq, dkdv)


@pytest.mark.parametrize("tq,tk,qo,d,fwd", [
    (16384, 16384, 0, 64, (8, 2, 1)),       # over the diagonal, 256 workgroups
    (16896, 16896, 67584, 64, (8, 1, 1)),   # all keys visible, more than a round
    (8192, 8192, 8192, 64, (8, 2, 1)),
    (1024, 1024, 1024, 64, (8, 4, 1)),      # too few keys for parts
    (1024, 1280, 4096, 64, (8, 2, 2)),
    (1024, 255, 4096, 64, (4, 1, 1)),
])
def test_pairs(tq, tk, qo, d, fwd):
    assert P.chunk_launch_shapes(tq, tk, qo, 0, 4, 4, d)["fwd_kernel"] == fwd


@pytest.mark.parametrize("rows,heads,d,alone,two", [
    # (forward, dQ, dK/dV groups of a fully visible pair) alone and two at a time:
    # groups go where two launches fill the chip without them
    (6144, 4, 128, (2, 2, 2), (2, 2, 2)),     # 96 workgroups
    (8192, 4, 128, (2, 2, 2), (1, 1, 1)),     # 128
    (39936, 4, 128, (2, 2, 2), (1, 1, 1)),    # 624
    (8192, 4, 64, (2, 2, 2), (2, 2, 2)),      # 128, but two to a CU
    (20480, 4, 64, (1, 1, 2), (1, 1, 1)),     # 320
])
def test_pairs_two_at_a_time(rows, heads, d, alone, two):
    for launches, expect in ((1, alone), (2, two)):
        got = P.chunk_launch_shapes(rows, rows, rows, 0, heads, heads, d, launches=launches)
        assert tuple(s[1] for s in got.values()) == expect, (launches, got)
        assert all(s[2] == 1 for s in got.values())


def test_diagonal_pair_keeps_its_groups():
    for launches in (1, 2):
        got = P.chunk_launch_shapes(16384, 16384, 16384, 16384, 4, 4, 128, launches=launches)
        assert {s[1] for s in got.values()} == {2}


def test_dq_takes_no_four_groups_on_more_than_half_the_chip():
    got = P.chunk_launch_shapes(19968, 19968, 0, 0, 2, 2, 128, causal=False)   # 156 workgroups
    assert got["bwd_dq_kernel"][1] < 4
    got = P.chunk_launch_shapes(1000, 900, 4096, 0, 4, 4, 128)                 # 32
    assert got["bwd_dq_kernel"][1] == 4
