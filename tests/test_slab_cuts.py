"""The slab schedule's ways to cut a convolution: each gives the bits of the fused and the tiled kernels."""
import re

import numpy as np
import pytest
import torch

from paper_2210_06223_amd import binding as B
from paper_2210_06223_amd import build, synth
from tests import _fake_hip as H
from tests import _util as U

# shape (N, H, W, C, M, S), listed or every cell, and the cuts (row blocks, waves, tiles per wave) that it selects: each
# instantiation at least once
CUTS = [
    ((1, 14, 14, 1024, 256, 1), True, ("1,2,1", "1,2,1", "1")),
    ((4, 14, 14, 1024, 256, 1), True, ("2,2,1", "1,2,1", "2")),
    ((8, 14, 14, 1024, 256, 1), True, ("2,4,1", "2,4,1", "2")),
    ((7, 14, 14, 1024, 256, 2), True, ("2,4,1", "2,2,1", "2")),
    ((13, 14, 14, 1024, 256, 2), True, ("2,4,2", "2,4,1", "4")),
    ((1, 50, 60, 1024, 256, 2), True, ("2,4,2", "2,4,1", "4")),
    ((2, 14, 14, 1024, 256, 7), True, ("1,2,1", "4,2,1", "1")),
    ((11, 14, 14, 1024, 256, 7), False, ("2,4,2", "4,4,1", "4")),
    ((25, 14, 14, 1024, 256, 7), False, ("2,4,2", "4,4,2", "4")),
    ((2, 7, 7, 2048, 512, 1), True, ("1,2,1", "1,2,1", "1")),
    ((7, 7, 7, 2048, 512, 1), True, ("2,2,1", "1,4,1", "2")),
    ((14, 7, 7, 2048, 512, 1), False, ("2,4,1", "1,4,2", "4")),
    ((1, 25, 42, 2048, 512, 1), True, ("2,4,2", "1,4,2", "4")),
]
CUT_IDS = ["x".join(map(str, c[0])) + ("" if c[1] else "_all") for c in CUTS]


def test_cuts_that_the_cases_select():
    """(Host only.)  The table above says what runs, and it names every slab kernel that the library holds."""
    got = H.run("result = [kernels(call('packed', BF16, *a, listed=l, flags=4)[1]) for a, l in %r]" % [(c[0], c[1]) for c in CUTS])
    seen = set()
    for (shape, _, cuts), names in zip(CUTS, got):
        C, M = shape[3:5]
        want = ["slab_conv1_kernel<%d,%d,%s>" % (C, M, cuts[0]), "slab_conv2_kernel<%d,%s>" % (M, cuts[1]),
                "slab_conv3_kernel<%d,%d,%s>" % (C, M, cuts[2])]
        assert [H.kernel_name(n) for n in names] == want, shape
        seen.update(want)
    held = set(re.findall(rb"_ZN6lasnet12_GLOBAL__N_1\d+slab_conv\d_kernelI[\w]*?EEv\w+", open(build.LIB, "rb").read()))
    assert {H.kernel_name(n.decode()) for n in held} == seen


@pytest.mark.gpu
@pytest.mark.parametrize("shape,listed,cuts", CUTS, ids=CUT_IDS)
def test_slab_bits_are_those_of_the_other_schedules(shape, listed, cuts):
    """The slab kernels sum in the order of the fused and the tiled ones, so the batch size, a capture or the entry that a call
    comes in by never shows in its output."""
    N, h, w, C, M, S = shape
    cfg = synth.BlockConfig("slab_bits", N, h, w, C, M, S, "bf16", 0.5, 94)
    d = U.dev_inputs(synth.make_block_inputs(cfg, want_f64=False))
    packed = B.lasnet_pack_weights(S, d["W1"], d["W2"], d["W3"])
    other = B.LASNET_FORCE_TILED if C == 2048 and h * w <= 49 else B.LASNET_FORCE_FUSED
    for r in (0.15, 0.6, 1.0) if listed else (None,):
        idx = count = None
        if listed:
            il = synth.make_index_list(N, cfg.G, cfg.GW, r, seed=N, order="shuffled")
            idx, count = U.list_tensor(il, cfg.P), torch.tensor([len(il)], dtype=torch.int32, device="cuda")
        outs = []
        for flags in (0, other):
            out = torch.full_like(d["x"], 777.0)
            B.lasnet_sparse_bottleneck_packed(d["x"], idx, count, S, M, packed, d["b1"], d["b2"], d["b3"], out=out,
                                              flags=flags | B.LASNET_POST_RELU)
            outs.append(U.bits(out))
        assert np.array_equal(outs[0], outs[1]), r


def test_where_the_slab_schedule_ends():
    """(Host only.)  The largest batch of each shape that takes it, and one image more."""
    ends = [((14, 14, 1024, 256, 1), 10), ((14, 14, 1024, 256, 2), 16), ((14, 14, 1024, 256, 7), 32), ((7, 7, 2048, 512, 1), 40)]
    got = H.run("result = [[['slab' in k for k in kernels(call('packed', BF16, n + e, *a, flags=4)[1])] for e in (0, 1)] for a, n in %r]" % ends)
    for (shape, _), (last, beyond) in zip(ends, got):
        assert all(last) and len(last) == 3 and not any(beyond), shape
