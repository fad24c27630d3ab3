"""The masker's cell kernel and the compaction at the edges of their work split: cells that just fit (or just do not fit)
the registers of 64 .. 1024 threads, runs of 1024 cells, more than 64 of them, a mask that is not aligned."""
import numpy as np
import pytest
import torch

from oracle import lasnet_oracle as O
from paper_2210_06223_amd import binding as B
from paper_2210_06223_amd import synth
from tests import _util as U

pytestmark = pytest.mark.gpu

CASES = [                                        # 16-byte pieces of a cell = S * S * C / (8 or 4)
    synth.BlockConfig("p1", 1, 3, 5, 8, 8, 1, "bf16", 0.5, 81),                 # one piece per cell
    synth.BlockConfig("p513_f32", 1, 3, 6, 228, 8, 3, "f32", 0.5, 82),          # 513: one more than 64 threads hold
    synth.BlockConfig("p8192", 1, 32, 64, 64, 8, 32, "bf16", 0.5, 83),          # the largest cell in registers
    synth.BlockConfig("p8256", 1, 32, 64, 64 + 8, 8, 32, "bf16", 0.5, 84),      # beyond it: the one-wave kernel
    synth.BlockConfig("cells1024", 1, 32, 32, 8, 8, 1, "bf16", 0.5, 85),        # one run of the compaction, exactly
    synth.BlockConfig("cells1025", 1, 25, 41, 8, 8, 1, "f32", 0.5, 86),         # and one cell more
    synth.BlockConfig("cells66000", 3, 200, 110, 8, 8, 1, "bf16", 0.5, 87),     # runs of several rounds
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
@pytest.mark.parametrize("shift", [0, 1])
def test_masker_and_list_edges(cfg, shift):
    inp = synth.make_block_inputs(cfg)
    d = U.dev_inputs(inp)
    k = int(round(cfg.r * cfg.P))
    bm = U.calibrate(inp, k)
    mask_o, idx_o, count_o, _ = O.masker(inp.f64["x"], inp.f64["Wm"], bm, cfg.S, 0.0)
    mask = torch.zeros(cfg.P + 16, dtype=torch.uint8, device="cuda")[shift:shift + cfg.P].view(cfg.N, cfg.G, cfg.GW)
    idx = torch.full((cfg.P,), -7, dtype=torch.int32, device="cuda")
    out = torch.full_like(d["x"], 768.0)
    _, _, count = B.lasnet_masker_ex(d["x"], d["Wm"], bm, cfg.S, 0.0, mask=mask, idx=idx, pass_out=out)
    torch.cuda.synchronize()
    assert int(count.item()) == count_o
    assert np.array_equal(mask.cpu().numpy(), mask_o)
    assert np.array_equal(idx.cpu().numpy()[:count_o], idx_o) and (idx.cpu().numpy()[count_o:] == -7).all()
    up = np.broadcast_to(O.upsample_mask(mask_o, cfg.S)[..., None].astype(bool), tuple(d["x"].shape))
    assert np.array_equal(U.bits(out)[~up], U.bits(d["x"])[~up])
    assert (U.to_f64(out)[up] == 768.0).all()
