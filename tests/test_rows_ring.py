"""Row schedule: rows through LDS rings with counted waits, against the build whose waits are for everything, bit for bit; and the zeros that
conv2 reads outside the image, in a workspace that holds anything.

What the comparison can show is a place overwritten before it was read, and a count too large for a reduction's first k-step or its ends: in the steady loop the
compiler's waits for the weights are for the next k-step's rows too."""
import numpy as np
import pytest
import torch

from paper_2210_06223_amd import binding as B
from paper_2210_06223_amd import build, synth
from tests import _util as U

pytestmark = pytest.mark.gpu

# one row block per wave with the reduction in one wave and over four, two blocks, and widths whose last k-step of conv1 is ragged (no ring there)
SHAPES = [(1, 24, 20, 256, 64, 4), (6, 28, 28, 1024, 32, 2), (1, 70, 75, 32, 256, 5), (1, 93, 99, 96, 250, 3), (3, 40, 40, 24, 256, 5), (17, 14, 14, 992, 200, 2)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_counted_waits_against_waits_for_everything(monkeypatch, shape, dtype):
    check = B.load_library(build.LIB_CHECK)
    cfg = synth.BlockConfig("ring", *shape, dtype, 0.5, 171)
    d = U.dev_inputs(synth.make_block_inputs(cfg, want_f64=False))
    for r in (0.1, 0.6, 1.0):
        il = synth.make_index_list(cfg.N, cfg.G, cfg.GW, r, seed=4)
        idx, count = U.list_tensor(il, cfg.P), torch.tensor([len(il)], dtype=torch.int32, device="cuda")
        outs = []
        for library in (B.lib(), check):
            monkeypatch.setattr(B, "_lib", library)
            outs.append(U.bits(B.lasnet_sparse_bottleneck(d["x"], idx, count, cfg.S, *U.weights(d))))
            monkeypatch.undo()
        assert np.array_equal(*outs), r


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_zeros_outside_the_image_whatever_the_workspace_holds(dtype):
    """A larger call leaves values of about 1e30 (its b1) where a smaller one's row of zeros is: the weights and the need bytes before y1 take
    the same room in both (16384 bytes hold either's), so that row is the larger one's pixel 800; 32 mid channels leave no padding in it.
    Against the scalar kernel, which has no workspace."""
    big = synth.BlockConfig("big", 9, 20, 20, 96, 32, 4, dtype, 1.0, 172)
    small = big.with_(N=2, name="small")
    db, ds = (U.dev_inputs(synth.make_block_inputs(c, want_f64=False)) for c in (big, small))
    want = B.lasnet_sparse_bottleneck(ds["x"], None, None, 4, *U.weights(ds), flags=B.LASNET_FORCE_GENERIC)
    db["b1"].fill_(1e30)
    B.lasnet_sparse_bottleneck(db["x"], None, None, 4, *U.weights(db))
    got = B.lasnet_sparse_bottleneck(ds["x"], None, None, 4, *U.weights(ds))
    U.assert_block_close(got, U.to_f64(want), ds["x"], np.ones(want.shape, bool), dtype)
