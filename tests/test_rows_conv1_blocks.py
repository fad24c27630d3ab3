"""Row schedule: the line from which conv1 of a long reduction takes two row blocks per wave."""
import numpy as np
import pytest
import torch

from paper_2210_06223_amd import binding as B
from paper_2210_06223_amd import synth
from tests import _fake_hip as H
from tests import _util as U
from tests.test_gpu_parity import _run_case

# (N, H, W, C, M, S) -> conv1's "row blocks, waves"
SHAPES = [
    ((12, 14, 14, 1024, 200, 2), "1,1"),       # 74 x 7 = 518 waves of two blocks
    ((17, 14, 14, 1024, 200, 2), "2,1"),       # 105 x 7
    ((17, 14, 14, 996, 200, 2), "2,1"),        # a ragged last k-step
    ((17, 14, 14, 992, 200, 2), "1,1"),        # 31 k-steps
    ((16, 14, 14, 1024, 288, 2), "1,1"),       # 98 x 3 workgroups
]


def test_cuts():
    """(Host only.)"""
    got = H.run("result = [[kernels(call('ex', d, *a, flags=4)[1]) for a in %r] for d in (F32, BF16)]" % [s[0] for s in SHAPES])
    for f, names in zip(("Fp32", "Bf16Wide"), got):
        for (shape, cut), call in zip(SHAPES, names):
            conv1 = [n for n in map(H.kernel_name, call) if "rows_conv1" in n]
            vec = shape[3] % (4 if f == "Fp32" else 8) == 0
            assert conv1 == ["rows_conv1_kernel<%s,%d,%s>" % (f, vec, cut)], (shape, f, conv1)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [s[0] for s in SHAPES[1:3]], ids=lambda s: "x".join(map(str, s)))
def test_two_blocks(shape, dtype):
    """Against the oracle; and the same bits as 12 images at a time, which one block per wave takes."""
    cfg = synth.BlockConfig("conv1_blocks", *shape, dtype, 0.4, 141)
    _run_case(cfg, k=int(round(cfg.r * cfg.P)))
    d = U.dev_inputs(synth.make_block_inputs(cfg, want_f64=False))
    w, x = U.weights(d), d["x"]
    whole = B.lasnet_sparse_bottleneck(x, None, None, cfg.S, *w, out=torch.empty_like(x))
    for part in (slice(0, 12), slice(5, 17)):
        xp = x[part].contiguous()
        out = B.lasnet_sparse_bottleneck(xp, None, None, cfg.S, *w, out=torch.empty_like(xp))
        assert np.array_equal(U.bits(out), U.bits(whole[part].contiguous()))
