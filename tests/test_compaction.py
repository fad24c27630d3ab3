"""The compaction's split into workgroups, at the edges of their runs."""
import numpy as np
import pytest
import torch

from oracle import lasnet_oracle as O
from paper_2210_06223_amd import binding as B
from paper_2210_06223_amd import synth
from tests import _fake_hip as H
from tests import _util as U


def test_small_workgroups_at_every_size():
    """(Host only.)  Runs of 1024 cells by four waves, at most 64 of them, then longer runs: a workgroup of 16 waves waits for
    room behind the masker of a large map (6272 cells: 1 to 2 us of the sequence)."""
    got = H.run("""
result = []
for cells in (1, 1024, 1025, 6272, 65536, 65537, 528000):
    F.fake_set(-1, 0, 0)
    x = T(vp(1 << 44).value, 1, 1, cells, 8, BF16)
    p = [vp((1 << 45) + i * (1 << 36)) for i in range(4)]
    L.lasnet_masker(ctypes.byref(x), p[0], ctypes.c_float(0), 1, ctypes.c_float(0), p[1], p[2], p[3], None)
    result.append([e[2:4] for e in (l.split() for l in F.fake_log().decode().splitlines()) if "compact" in e[1]][0])
""")
    assert got == [[n, "256"] for n in ("1", "1", "2", "7", "64", "33", "58")]


@pytest.mark.gpu
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("N,h,w", [(1, 64, 128), (1, 1, 8193), (3, 400, 440)], ids=["8192", "8193", "528000"])
def test_compaction_edges(N, h, w, shift):
    """Whole runs, one cell more, and runs of nine rounds; a mask that is not aligned."""
    cfg = synth.BlockConfig("compact", N, h, w, 8, 8, 1, "bf16", 0.5, 101)
    inp = synth.make_block_inputs(cfg)
    d = U.dev_inputs(inp)
    bm = U.calibrate(inp, cfg.P // 2)
    mask_o, idx_o, count_o, _ = O.masker(inp.f64["x"], inp.f64["Wm"], bm, 1, 0.0)
    mask = torch.zeros(cfg.P + 16, dtype=torch.uint8, device="cuda")[shift:shift + cfg.P].view(N, h, w)
    idx = torch.full((cfg.P,), -7, dtype=torch.int32, device="cuda")
    _, _, count = B.lasnet_masker(d["x"], d["Wm"], bm, 1, 0.0, mask=mask, idx=idx)
    got = idx.cpu().numpy()
    assert int(count.item()) == count_o and np.array_equal(mask.cpu().numpy(), mask_o)
    assert np.array_equal(got[:count_o], idx_o) and (got[count_o:] == -7).all()
