"""The branches that a call's sizes choose between, each at the sizes where it can go wrong, against the CPU oracle
(bit-exact but for the float32 advantages: float64 arithmetic on both sides, see test_gpu_parity)."""
import numpy as np
import pytest

from test_gpu_parity import _custom, check_gather_advantage, check_scatter, check_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("length", [341, 256, 205, 204, 22, 21, 17, 16, 15, 4, 3])
def test_slots_of_a_granule(length):
    """Equal lengths round the counts at which a 1024-token granule changes its path: 4 slots (its record holds them), 5 (a
    wave stages them), 47 and 48, 63 and 64 (one pass or two over the staged slots), more slots than 16-byte chunks."""
    n = max(64, 9000 // length) // 32 * 32
    lens = np.full(n, length, np.int32)
    lens[::7] += np.arange(len(lens[::7])) % 3
    for align in (1, 5):
        w = _custom(lens, 4, 4, 4096, n_src=2, seed=length)
        check_step(w, align=align, label=f"length {length}", two_calls=True)
        check_gather_advantage(w, align=align, label=f"length {length}")
    check_scatter(_custom(lens, 4, 4, 4096, n_src=2, seed=length), label=f"length {length}")
