"""Row schedule: reductions of every length around the rings of two and three k-steps, so that each of the GEMM's straight-line ends runs (one
to five k-steps; whole rounds and each of these), in one wave and shared by four (some of whose shares are empty)."""
import pytest

from paper_2210_06223_amd import synth
from tests import _fake_hip as H
from tests.test_gpu_parity import _run_case

# (C, M): k-steps of conv1 / of a tap of conv2 and of conv3 1/1, 2/2, 3/3, 4/4, 5/5 (ragged), and 8 to 12 for conv1, which four waves share
WIDTHS = [(32, 16), (64, 40), (96, 72), (128, 104), (132, 136), (256, 24), (292, 40), (320, 72), (352, 100), (384, 136)]
CASES = [(c, m, dt) for c, m in WIDTHS for dt in ("f32", "bf16")]
SHAPE = (4, 24, 20)                                          # with S = 4: 120 cells


def test_the_row_schedule_runs_them():
    """(Host only.)"""
    got = H.run("result = [kernels(call('ex', {'f32': F32, 'bf16': BF16}[d], *%r, c, m, 4, flags=4)[1]) for c, m, d in %r]" % (SHAPE, CASES))
    shared = set()
    for case, names in zip(CASES, got):
        names = [H.kernel_name(n) for n in names if "rows_conv" in n]
        assert len(names) == 3, case
        shared.update((n[:10], n.endswith(",4>")) for n in names)
    assert {("rows_conv1", True), ("rows_conv1", False), ("rows_conv2", True), ("rows_conv3", False)} <= shared


@pytest.mark.gpu
@pytest.mark.parametrize("C,M,dtype", CASES, ids=lambda v: str(v))
def test_reductions_of_every_length(C, M, dtype):
    cfg = synth.BlockConfig("ends", *SHAPE, C, M, 4, dtype, 0.4, 151)
    _run_case(cfg, k=48)
    _run_case(cfg, k=cfg.P)
