"""The row schedule's map of needed pixels from long lists: scattered entry by entry, against scanned by the plan."""
import pytest
import torch

from paper_2210_06223_amd import binding as B
from paper_2210_06223_amd import synth
from tests import _fake_hip as H
from tests import _util as U
from tests.test_gpu_parity import _run_case

CASES = [
    synth.BlockConfig("p1024_f32", 1, 32, 32, 20, 40, 1, "f32", 0.1, 111),          # the longest list that is scanned
    synth.BlockConfig("p1025_f32", 1, 25, 41, 20, 40, 1, "f32", 0.1, 112),
    synth.BlockConfig("p1190_s3_bf16", 2, 51, 105, 33, 20, 3, "bf16", 0.05, 113),   # windows of 5 rows, odd map
    synth.BlockConfig("p1152_s7_f32", 32, 42, 42, 16, 12, 7, "f32", 0.03, 114),     # many images, few patches
]


def test_which_lists_are_scattered():
    """(Host only.)  And the plan's workgroups do not scan those: 64 workgroups that each walk 1.6 M entries took 12 ms."""
    got = H.run("result = [[k for k in kernels(call('ex', {'f32': F32, 'bf16': BF16}[d], *a)[1])] for d, a in %r]"
                % [(c.dtype, (c.N, c.H, c.W, c.C, c.M, c.S)) for c in CASES])
    for cfg, names in zip(CASES, got):
        names = [H.kernel_name(n).split("<")[0] for n in names]
        assert names == ["copy_kernel", "rows_plan_kernel"] + ["rows_need_kernel"] * (cfg.P > 1024) + ["rows_conv%d_kernel" % i for i in (1, 2, 3)], cfg


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_long_lists(cfg):
    _run_case(cfg, k=int(round(cfg.r * cfg.P)))
    _run_case(cfg, k=cfg.P)
    _run_case(cfg, k=0)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("S,count", [(2, -10**9), (2, -1), (3, -2**31), (5, -(2**31) // 25 - 7)])
def test_a_negative_count_is_an_empty_list(dtype, S, count):
    """Also one that, times S * S, wraps to a positive number of rows in 32 bits (-10**9 * 4 = 294967296 there)."""
    cfg = synth.BlockConfig("negative", 1, 6 * S, 4 * S, 64, 40, S, dtype, 0.5, 115)
    d = U.dev_inputs(synth.make_block_inputs(cfg, want_f64=False))
    idx = torch.arange(cfg.P, dtype=torch.int32, device="cuda")
    out = torch.full_like(d["x"], 777.0)
    B.lasnet_sparse_bottleneck(d["x"], idx, torch.tensor([count], dtype=torch.int32, device="cuda"), S, *U.weights(d), out=out)
    assert (U.bits(out) == U.bits(d["x"])).all()
