"""Which calls without a matrix-core kernel of their own run the row schedule, and which the scalar kernel (host only)."""
import pytest

from tests import _fake_hip as H

# (N, H, W, C, M, S) -> the scalar kernel is the faster one (measured: times beside the rule)
CASES = [
    ((1, 8, 8, 16, 4, 2), True), ((1, 1, 1, 1, 1, 1), True), ((1, 28, 28, 32, 8, 2), True), ((4, 28, 28, 32, 8, 4), True),
    ((16, 28, 28, 16, 4, 2), True), ((64, 28, 28, 16, 4, 7), True), ((64, 112, 112, 16, 4, 7), True), ((256, 28, 28, 16, 4, 4), True),
    ((64, 28, 28, 8, 2, 4), True),
    ((1, 8, 8, 48, 12, 4), False), ((16, 28, 28, 32, 8, 2), False), ((64, 28, 28, 64, 4, 4), False), ((64, 112, 112, 16, 4, 2), False),
    ((64, 112, 112, 32, 8, 4), False), ((64, 28, 28, 16, 4, 1), False), ((1, 56, 56, 256, 64, 4), False),
    ((16, 14, 14, 1024, 256, 2), False), ((13, 28, 20, 192, 48, 4), False),
]


@pytest.mark.parametrize("dtype", ["F32", "BF16"])
def test_little_work_stays_on_one_launch(dtype):
    got = H.run("result = [[st, kernels(ev)] for st, ev in [call('ex', %s, *a, flags=4 | 2) for a in %r]]" % (dtype, [c[0] for c in CASES]))
    for (shape, scalar), (st, names) in zip(CASES, got):
        assert st == 0 and (H.kernel_name(names[-1]).split("<")[0] == "bneck_generic_kernel") == scalar, (shape, names)
