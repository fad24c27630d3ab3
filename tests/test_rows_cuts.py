"""The row schedule's ways to cut a convolution (row blocks per wave, waves per tile's reduction), each against the oracle, with
ragged last tiles and groups, with 16-byte and with element-wise loads, and with needed pixels that are few or all."""
import re

import pytest

from paper_2210_06223_amd import build, synth
from tests import _fake_hip as H
from tests.test_gpu_parity import _run_case

from paper_2210_06223_amd import binding as B

# (N, H, W, C, M, S) and the cuts "row blocks, waves" of conv1, conv2 and conv3, the same in both types
CUTS = [
    ((16, 32, 32, 24, 256, 4), ("4,1", "4,1", "1,4")),
    ((6, 28, 28, 1024, 32, 2), ("1,4", "1,4", "4,1")),
    ((1, 93, 99, 33, 250, 3), ("4,1", "2,1", "1,4")),
    ((1, 54, 54, 1000, 40, 2), ("1,4", "1,4", "2,1")),
    ((1, 70, 75, 21, 256, 5), ("2,1", "1,1", "1,4")),
    ((1, 28, 26, 1001, 40, 2), ("1,4", "1,4", "1,1")),
    ((3, 14, 7, 40, 20, 7), ("1,1", "1,4", "1,1")),
    ((2, 42, 49, 1001, 33, 7), ("1,4", "1,4", "4,1")),
    ((5, 42, 49, 24, 250, 7), ("4,1", "2,1", "1,4")),
    ((1, 54, 54, 1003, 40, 2), ("1,4", "1,4", "2,1")),
    ((3, 40, 40, 24, 256, 5), ("2,1", "1,1", "1,4")),
    ((16, 32, 32, 21, 256, 4), ("4,1", "4,1", "1,4")),
    ((3, 14, 7, 39, 20, 7), ("1,1", "1,4", "1,1")),
]
CASES = [(synth.BlockConfig("rows_%s_%s" % ("x".join(map(str, a)), dt), *a, dt, 0.3, 120 + i), cuts)
         for i, (a, cuts) in enumerate(CUTS) for dt in ("f32", "bf16")]


def test_cuts_that_the_cases_select():
    """(Host only.)  The table above says what runs, and it names every row kernel that the library holds."""
    got = H.run("result = [kernels(call('ex', {'f32': F32, 'bf16': BF16}[d], *a, flags=4)[1]) for d, a in %r]"
                % [(c.dtype, (c.N, c.H, c.W, c.C, c.M, c.S)) for c, _ in CASES])
    seen = set()
    for (cfg, cuts), names in zip(CASES, got):
        names = [H.kernel_name(n) for n in names if "rows_conv" in n]
        f, vec = ("Fp32", cfg.C % 4 == 0) if cfg.dtype == "f32" else ("Bf16Wide", cfg.C % 8 == 0)
        assert names == ["rows_conv1_kernel<%s,%d,%s>" % (f, vec, cuts[0]), "rows_conv2_kernel<%s,%s>" % (f, cuts[1]),
                         "rows_conv3_kernel<%s,%d,%s>" % (f, vec, cuts[2])], cfg
        seen.update(names)
    held = set(re.findall(rb"_ZN6lasnet12_GLOBAL__N_1\d+rows_conv\d_kernelI[\w]*?EEv\w+", open(build.LIB, "rb").read()))
    held = {H.kernel_name(n.decode()) for n in held}
    assert held == seen, held ^ seen


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,cuts", CASES, ids=[c.name for c, _ in CASES])
def test_row_cuts_match_the_oracle(cfg, cuts):
    _run_case(cfg, k=max(1, int(round(cfg.r * cfg.P))))
    _run_case(cfg, k=max(1, cfg.P // 50), flags=B.LASNET_POST_RELU)
