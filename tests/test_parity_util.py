"""The parity checks themselves: what they must and must not let through."""
import numpy as np
import pytest

from oracle import attention as ora
from paper_2511_13198_amd import workloads as wl
from tests import parity_util as pu


def _gradients(lengths, d=64):
    cu = wl.cu_from_lengths(lengths)
    bits = wl.host_inputs(sum(lengths), 2, 1, d, seed=5)
    f = {n: wl.bf16_bits_to_f64(b) for n, b in bits.items()}
    return cu, ora.backward(f["q"], f["k"], f["v"], f["do"], cu, True, d ** -0.5)


def test_lost_late_key_tile_fails_the_block_check():
    """The gradients of the last 64 keys of a causal sequence, zeroed: within
    the bound on the whole tensor, found by the check in blocks."""
    cu, (_, _, _, dk, dv) = _gradients([6208])
    for name, ref in (("dK", dk), ("dV", dv)):
        got = ref.copy()
        got[6144:] = 0.0
        rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        assert rel < pu.REL_L2
        with pytest.raises(AssertionError, match="rows from 6144"):
            pu.check_blocks(name, got, ref, cu)


@pytest.mark.parametrize("row,head", [(0, 0), (700, 1), (1023, 0), (1087, 1)])
def test_block_check_places_a_lost_tile(row, head):
    """One head's block of one of several segments, the ragged last one too."""
    cu, (o, _, dq, _, _) = _gradients([1000, 0, 88, 7])
    for name, ref in (("O", o), ("dQ", dq)):
        assert pu.check_blocks(name, ref * (1 + 2e-3), ref, cu) < 3e-3
        got = ref.copy()
        seg = max(a for a in cu if a <= row)
        a = seg + (row - seg) // 64 * 64
        got[a:min(a + 64, 1088), head] = 0.0
        with pytest.raises(AssertionError, match=f"head {head}"):
            pu.check_blocks(name, got, ref, cu)
