"""Infinite weights, y values and maps in the row schedule: the infinities and NaNs of the same sums in fp32."""
import pytest
import torch

from paper_2210_06223_amd import binding as B
from paper_2210_06223_amd import synth
from tests import _util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("where", ["W2", "W3", "W2_W3", "W1", "x"])
def test_infinities_match_the_scalar_kernel(dtype, where):
    """Products of an infinity with a positive y are infinite and with a zero y NaN (which a ReLU makes 0), whichever kernel
    forms them; finite results agree to the tolerance of either."""
    cfg = synth.BlockConfig("infinite", 2, 8, 12, 40, 33, 4, dtype, 0.5, 151)
    d = U.dev_inputs(synth.make_block_inputs(cfg, want_f64=False))
    inf = float("inf")
    d["W1"][:, :20] = torch.sign(d["W1"][:, :20].float()).to(d["W1"].dtype)             # y values of few bits among the others
    if "W2" in where:
        d["W2"].view(33, 3, 3, 33)[3, 1, 1, 5] = inf
        d["W2"].view(33, 3, 3, 33)[4, 0, 2, 6] = -inf
    if "W3" in where:
        d["W3"].view(40, 33)[7, 9] = inf
        d["W3"].view(40, 33)[8, 10] = -inf
    if where == "W1":
        d["W1"].view(33, 40)[11, 2] = inf
    if where == "x":
        d["x"][0, 3, 5, 2] = inf
    il = synth.make_index_list(cfg.N, cfg.G, cfg.GW, 0.7, seed=2)
    idx, count = U.list_tensor(il, cfg.P), torch.tensor([len(il)], dtype=torch.int32, device="cuda")
    rows = B.lasnet_sparse_bottleneck(d["x"], idx, count, cfg.S, *U.weights(d)).double()
    scalar = B.lasnet_sparse_bottleneck_noalloc(d["x"], idx, count, cfg.S, *U.weights(d), out=torch.empty_like(d["x"])).double()
    assert torch.isinf(scalar).any()
    for kind in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(kind(rows), kind(scalar)), kind
    ok = torch.isfinite(scalar)
    assert (rows - scalar)[ok].abs().max() <= (2.0 ** -8 if dtype == "bf16" else 1e-5) * scalar[ok].abs().max()
