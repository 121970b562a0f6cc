"""Key groups (forward, dQ) and query groups (dK/dV): workgroups of small
launches whose waves share the rows (keys) and split the inner loop, combined in
LDS.  Every element against the fp64 oracle at the sizes where the groups begin,
end or leave waves without work, each case with the shapes that it is there for
(waves, groups, parts); the same results from a workspace that only
holds the launch without groups and parts."""
import numpy as np
import pytest

from oracle import attention as ora
from paper_2511_13198_amd import workloads as wl
from tests.parity_util import check_close, log, to_device_bf16
from tests.test_gpu_chunks import _check_partial, _dev, _host
from tests.test_gpu_parity import _full_parity

pytestmark = pytest.mark.gpu


def _shapes(lengths, hq, hkv, d, causal):
    """(waves, groups, parts) of the forward, dQ and dK/dV launches."""
    from paper_2511_13198_amd import pdyattn
    got = pdyattn.launch_shapes(sum(lengths), len(lengths), max(lengths), hq, hkv, d, causal)
    return [got[n] for n in ("fwd_kernel", "bwd_dq_kernel", "bwd_dkdv_kernel")]


# (lengths, hq, hkv, d, causal, the launches' shapes)
GROUP_CASES = [
    # one row, one key
    ([1], 1, 1, 64, True, [(4, 1, 1), (4, 1, 1), (8, 2, 1)]),
    ([65], 3, 1, 128, True, [(4, 1, 1), (4, 1, 1), (8, 2, 6)]),
    # from 256 keys on four groups; five 64-row tiles and one row
    ([255], 3, 1, 128, True, [(4, 1, 1), (4, 1, 1), (8, 2, 12)]),
    ([256], 3, 1, 128, True, [(8, 4, 1), (8, 4, 1), (8, 2, 12)]),
    ([321], 3, 1, 64, True, [(8, 4, 1), (8, 4, 1), (8, 1, 9)]),
    # four groups, unsplit
    ([512], 8, 8, 64, True, [(8, 4, 1), (8, 4, 1), (8, 2, 3)]),
    ([511], 2, 2, 128, False, [(8, 4, 1), (4, 1, 4), (8, 2, 2)]),
    # two groups, balanced parts, one row in the last tile
    ([2049], 1, 1, 128, True, [(8, 1, 9), (8, 2, 9), (8, 2, 11)]),
    ([2049], 2, 2, 128, True, [(8, 2, 9), (8, 2, 9), (8, 2, 11)]),
    # three query heads per key head
    ([2500], 6, 2, 64, True, [(8, 2, 3), (8, 2, 3), (8, 1, 15)]),
    ([2500], 6, 2, 128, True, [(8, 2, 3), (8, 2, 3), (8, 2, 11)]),
    # uniform parts: one group, and two
    ([2304], 2, 1, 128, False, [(8, 1, 4), (8, 1, 4), (8, 1, 4)]),
    ([2304], 4, 4, 128, False, [(8, 2, 2), (8, 2, 2), (8, 2, 2)]),
    # packed: dK/dV over 128-key tiles
    ([600, 1, 129, 1024] * 4, 3, 3, 128, True, [(4, 1, 1), (4, 1, 1), (8, 2, 1)]),
    ([2048, 1000, 2000], 4, 2, 128, True, [(4, 1, 2), (4, 1, 2), (8, 1, 4)]),
    ([1800, 1700, 1500], 4, 4, 128, True, [(4, 1, 1), (4, 1, 2), (8, 2, 2)]),
    ([103, 52] * 5, 32, 8, 64, True, [(4, 1, 1), (4, 1, 1), (8, 2, 2)]),
    ([300, 1, 129, 512], 2, 1, 64, True, [(4, 1, 1), (4, 1, 1), (8, 1, 4)]),
    ([300, 0, 127], 4, 4, 128, False, [(4, 1, 1), (4, 1, 1), (8, 2, 1)]),
    # d = 64: 300 8-wave tiles, so a 4-wave forward
    ([2305], 30, 15, 64, True, [(4, 1, 1), (8, 1, 2), (8, 2, 2)]),
    # the same, packed: 4-wave forward and dQ
    ([2100, 65], 30, 30, 64, True, [(4, 1, 1), (4, 1, 1), (8, 1, 1)]),
    # 4-wave query tiles in uniform parts
    ([10153], 2, 1, 64, True, [(4, 1, 4), (4, 1, 4), (8, 1, 12)]),
]


@pytest.mark.parametrize("lengths,hq,hkv,d,causal,shapes", GROUP_CASES)
def test_groups_full_parity(lengths, hq, hkv, d, causal, shapes):
    assert _shapes(lengths, hq, hkv, d, causal) == shapes
    _full_parity(lengths, hq, hkv, d, causal)


@pytest.mark.parametrize("lengths,hq,hkv,d,causal", [
    # short segments that fill the chip: 4-wave dK/dV workgroups of 128 keys
    ([127, 128, 129, 1, 0, 257, 33, 31] * 4, 24, 12, 128, True),
    ([127, 128, 129, 1, 0, 257, 33, 31] * 4, 16, 16, 64, False),
    ([1, 2, 3, 32, 64, 65] * 6, 64, 16, 128, False),
])
def test_short_segments_full_parity(lengths, hq, hkv, d, causal):
    assert _shapes(lengths, hq, hkv, d, causal) == [(4, 1, 1)] * 3
    _full_parity(lengths, hq, hkv, d, causal)


@pytest.mark.parametrize("nseg,hi,rest,hq,d,scheduled", [
    # segment-major: to 64 segments and 16,384 segments x workgroups
    (2, 4000, 4000, 1, 128, False), (48, 1100, 100, 2, 64, False), (65, 1100, 100, 2, 64, True),
    (64, 1100, 100, 2, 64, True),    # dK/dV in two parts of 128-key tiles beyond them
    (64, 1100, 1100, 2, 64, True),
    (48, 2841, 1300, 1, 64, True),   # within them but for its parts
    # level-major: to 128 segments
    (63, 500, 500, 2, 128, False), (128, 500, 500, 1, 64, False), (129, 500, 500, 1, 64, True),
])
def test_packed_placement(nseg, hi, rest, hq, d, scheduled):
    """Packed batches on both sides of the sizes up to which the workgroups
    place their items themselves: every element (an item placed twice, wrongly
    or not at all shows), equal counts and empty segments among them, and the
    schedule kernel runs only beyond."""
    from paper_2511_13198_amd import pdyattn
    rng = np.random.default_rng(nseg)
    lengths = [int(x) for x in rng.integers(1, rest + 1, size=nseg)]
    lengths[0] = hi                    # the longest, so that the order is known
    lengths[-1] = 0
    if nseg > 2:
        lengths[1] = lengths[2]
    pdyattn.profile_start()
    _full_parity(lengths, hq, hq, d, True)
    ran = "plan_kernel" in pdyattn.profile_stop()
    assert ran == scheduled


@pytest.mark.parametrize("nseg,hq,hkv,d,causal", [
    (300, 1, 1, 128, True),   # 44 workgroups over the 8 XCDs of one head
    (131, 2, 2, 64, False),   # 3 of each of two heads over 4 XCDs
    (67, 4, 4, 64, True),     # 3 of each of four heads over 2 XCDs
    (33, 8, 4, 128, True),    # one of each of eight heads
    (200, 3, 3, 64, True),    # heads that do not divide the XCDs
])
def test_last_partial_round(nseg, hq, hkv, d, causal):
    """One workgroup per segment and head, a full round and a ragged rest: every
    item has its place (one left out keeps the NaN it was given, one of
    accumulating launches taken twice would not match)."""
    assert nseg * hq > 256 and nseg * hq % 256
    _full_parity([64 + (i * 7) % 60 for i in range(nseg)], hq, hkv, d, causal)


def test_last_partial_round_single():
    """dQ and dK/dV over 127 tiles of 128 rows, two XCDs per head: the second round
    is four workgroups short."""
    from tests.test_gpu_parity import _sampled_parity
    w = wl.Workload("single16200_h4", [16200], 4, 4, 128)
    assert _shapes([16200], 4, 4, 128, True)[1:] == [(8, 2, 1)] * 2
    _sampled_parity(w, device_gen=True, heads=[0, 3], kv_heads=[1, 2], per_seg_random=48,
                    tail_cols=128)


PAIRS = [
    # (T, hq, hkv, d, causal, (qa, qb), (ka, kb), shapes); the diagonal, an
    # earlier, a later and an overlapping key chunk, ragged ends, over and under
    # 2,048 rows
    (4700, 1, 1, 128, True, (2400, 4700), (0, 2399), [(8, 2, 4)] * 3),
    (2305, 1, 1, 128, True, (0, 2305), (0, 2305), [(8, 2, 4)] * 3),
    (4600, 2, 1, 64, True, (2300, 4600), (2300, 4600), [(8, 2, 4)] * 3),
    (3000, 1, 1, 128, True, (100, 2500), (1700, 3000), [(8, 2, 2), (8, 2, 2), (8, 2, 4)]),
    (900, 3, 1, 128, True, (200, 765), (0, 566), [(8, 4, 1), (8, 4, 1), (8, 2, 4)]),
    (1300, 2, 2, 64, False, (0, 1), (1, 1300), [(8, 2, 2), (8, 2, 2), (8, 2, 1)]),
    # nothing visible
    (2700, 1, 1, 64, True, (0, 300), (300, 2700), [(8, 2, 4), (8, 2, 4), (8, 1, 1)]),
    (10000, 4, 4, 128, True, (8192, 8256), (0, 8192), [(8, 2, 4), (8, 2, 4), (8, 2, 1)]),
]


@pytest.mark.parametrize("T,hq,hkv,d,causal,qs,ks,shapes", PAIRS)
def test_group_pairs(T, hq, hkv, d, causal, qs, ks, shapes):
    """Partial forward, the pair's gradients, and both again from the smallest
    accepted workspace and added to what the gradients hold."""
    import torch
    from paper_2511_13198_amd import pdyattn
    bits, f = _host(T, hq, hkv, d, 23)
    scale = 1.0 / np.sqrt(d)
    (qa, qb), (ka, kb) = qs, ks
    tq, tk = qb - qa, kb - ka
    got = pdyattn.chunk_launch_shapes(tq, tk, qa, ka, hq, hkv, d, causal)
    assert [got[n] for n in ("fwd_kernel", "bwd_dq_kernel", "bwd_dkdv_kernel")] == shapes
    log(f"  T={T} chunk q[{qa},{qb}) k[{ka},{kb}) Hq={hq} Hkv={hkv} d={d} causal={causal}")
    o_ref, l_ref = ora.partial_forward(f["q"][qa:qb], f["k"][ka:kb], f["v"][ka:kb], qa, ka,
                                       causal, scale)
    q, do = _dev(bits, "q", qa, qb), _dev(bits, "do", qa, qb)
    k, v = _dev(bits, "k", ka, kb), _dev(bits, "v", ka, kb)
    # schedule space (unused) and D, no partial results
    small = 4096 + 4 * hq * tq + 64 * (tq + tk)
    ws = [None, torch.empty(small, dtype=torch.uint8, device="cuda")]
    for w in ws:
        o = torch.full_like(q, float("nan"))
        lse = torch.full((hq, tq), float("nan"), dtype=torch.float32, device=q.device)
        pdyattn.attn_fwd_chunk(q, k, v, qa, ka, causal, scale, out=o, lse=lse, workspace=w)
        torch.cuda.synchronize()
        _check_partial("O", "LSE", o.double().cpu().numpy(), lse.cpu().numpy(), o_ref, l_ref)
    O, L = ora.forward(f["q"], f["k"], f["v"], np.array([0, T]), causal, scale)
    o_bits = wl.f32_to_bf16_bits(O[qa:qb].astype(np.float32))
    l32 = np.ascontiguousarray(L[:, qa:qb].astype(np.float32))
    ref = ora.partial_backward(f["q"][qa:qb], f["k"][ka:kb], f["v"][ka:kb],
                               wl.bf16_bits_to_f64(o_bits), l32.astype(np.float64), f["do"][qa:qb],
                               qa, ka, causal, scale)
    o_d, l_d = to_device_bf16(o_bits), torch.from_numpy(l32).cuda()
    for w, add in ((None, False), (ws[1], False), (None, True)):
        g = [torch.full(s, 0.5 if add else float("nan"), dtype=torch.float32, device="cuda")
             for s in ((tq, hq, d), (tk, hkv, d), (tk, hkv, d))]
        pdyattn.attn_bwd_chunk(q, k, v, o_d, l_d, do, qa, ka, causal, scale, dq=g[0], dk=g[1],
                               dv=g[2], workspace=w, accumulate=add)
        torch.cuda.synchronize()
        for nm, got, r in zip(("dQc", "dKc", "dVc"), g, ref):
            got = got.double().cpu().numpy() - (0.5 if add else 0.0)
            if not np.any(r):
                assert not np.any(got), f"{nm}: nonzero gradient for an invisible pair"
            else:
                check_close(nm, got, r)


@pytest.mark.parametrize("value", [float("nan"), 3e38, -3e38])
@pytest.mark.parametrize("T,hq,hkv,d,causal,chunk,shape", [
    (300, 4, 4, 128, True, None, (8, 4, 1)),
    (512, 8, 8, 64, True, None, (8, 4, 1)),
    (2049, 2, 2, 128, True, None, (8, 2, 9)),     # two groups, balanced parts
    (511, 2, 2, 128, False, None, (8, 4, 1)),
    (700, 1, 1, 64, False, None, (8, 4, 1)),
    (2304, 4, 2, 128, False, None, (8, 2, 2)),    # two groups, uniform parts
    (2600, 6, 6, 64, True, None, (4, 1, 4)),      # one group, parts
    (2100, 30, 30, 64, True, None, (4, 1, 1)),    # one group, no parts
    (2305, 1, 1, 128, True, (2305, 2305), (8, 2, 4)),
    (565, 3, 1, 128, True, (565, 565), (8, 4, 1)),
])
def test_nonfinite_logits(value, T, hq, hkv, d, causal, chunk, shape):
    """One key of NaN, or one whose logits overflow (queries made positive), seen
    by one part or group of a row only: a row that sees a NaN or +inf logit has
    O = NaN and LSE = -inf in every launch shape, a key of -inf logits weighs
    nothing, and the rows before it are untouched."""
    import torch
    from paper_2511_13198_amd import pdyattn
    name = "fwd_kernel"
    got = (pdyattn.chunk_launch_shapes(T, T, 0, 0, hq, hkv, d, causal) if chunk else
           pdyattn.launch_shapes(T, 1, T, hq, hkv, d, causal))[name]
    assert got == shape
    bits, f = _host(T, hq, hkv, d, 29)
    j, scale = T // 3, 1.0 / np.sqrt(d)
    f["q"] = np.abs(f["q"])
    kd = torch.from_numpy(f["k"]).to(torch.bfloat16)
    kd[j] = value
    q = _dev(bits, "q", 0, T).abs()
    k, v = kd.cuda(), _dev(bits, "v", 0, T)
    o = torch.zeros_like(q)
    lse = torch.zeros((hq, T), dtype=torch.float32, device="cuda")
    if chunk:
        pdyattn.attn_fwd_chunk(q, k, v, 0, 0, causal, scale, out=o, lse=lse)
    else:
        cu = torch.tensor([0, T], dtype=torch.int32, device="cuda")
        pdyattn.attn_fwd(q, k, v, cu, T, causal, scale, out=o, lse=lse)
    torch.cuda.synchronize()
    keep = np.arange(T) != j
    if value < 0:  # as if the key were not there (row j sees the keys before it)
        cut = {n: f[n][keep] for n in ("k", "v")}
        ro, rl = ora.partial_forward(f["q"][:j], cut["k"], cut["v"], 0, 0, causal, scale)
        # a later row i sees the kept keys 0 .. i - 1
        so, sl = ora.partial_forward(f["q"][j:], cut["k"], cut["v"], j - 1, 0, causal, scale)
        check_close("O", o.double().cpu().numpy(), np.concatenate([ro, so]))
        check_close("LSE", lse.cpu().numpy(), np.concatenate([rl, sl], axis=1))
        return
    first = j if causal else 0
    assert torch.isnan(o[first:]).all()
    assert torch.isneginf(lse[:, first:]).all()
    if first:
        ro, rl = ora.partial_forward(f["q"][:j], f["k"][:j], f["v"][:j], 0, 0, causal, scale)
        check_close("O", o[:j].double().cpu().numpy(), ro)
        check_close("LSE", lse[:, :j].cpu().numpy(), rl)


def test_underfilled_pairs_split():
    """A pair whose workgroups fill less than half the chip takes partial
    results; one that fills it, and any pair in a small workspace, does not."""
    import torch
    from paper_2511_13198_amd import pdyattn
    for t, h, expect in ((4096, 1, True), (8192, 4, False)):
        x = wl.device_inputs(t, h, h, 128, seed=3)
        pdyattn.profile_start()
        pdyattn.attn_fwd_chunk(x["q"], x["k"], x["v"], t, 0)
        got = "split_merge_kernel" in pdyattn.profile_stop()
        assert got == expect
        ws = torch.empty(1 << 16, dtype=torch.uint8, device="cuda")
        pdyattn.profile_start()
        pdyattn.attn_fwd_chunk(x["q"], x["k"], x["v"], t, 0, workspace=ws)
        assert "split_merge_kernel" not in pdyattn.profile_stop()
