"""How the fused and the streaming kernel cut the list into runs and decode its cells: every cut gives every listed patch the same bits."""
import numpy as np
import pytest
import torch

from oracle import lasnet_oracle as O
from paper_2210_06223_amd import binding as B
from paper_2210_06223_amd import synth
from tests import _util as U

pytestmark = pytest.mark.gpu

# Lists of one entry, of a few more and less than the chip's workgroups, of several rounds with runs of two lengths, and of
# patches apart from each other (a batch that exceeds the y1 rows is cut and runs again).  Maps with one column or one row of
# cells (a divisor of one) and with sides that are no powers of two.
CASES = [
    # the last list with one run per CU and the first with one per place of a workgroup
    (16, 28, 28, 512, 128, 4, (640, 641, 768, 769)),
    (10, 28, 28, 512, 128, 2, (1792, 1793)),
    (4, 28, 28, 512, 128, 1, (3072, 3073)),
    (1, 56, 56, 256, 64, 1, (3072, 3073)),
    (2, 56, 56, 256, 64, 2, (1024, 1025)),
    (6, 56, 56, 256, 64, 2, (1, 255, 511, 513, 4095, 4097, 4600)),
    (3, 12, 84, 256, 64, 4, (1, 9, 63, 180)),
    (40, 8, 2, 512, 128, 2, (3, 100, 159)),
    (7, 3, 33, 512, 128, 1, (17, 300, 693)),
    (2, 14, 63, 512, 128, 7, (1, 20, 36)),
    (41, 2, 46, 1024, 256, 2, (7, 256, 257, 900)),
    (5, 45, 3, 1024, 256, 1, (64, 600)),
    (17, 56, 56, 256, 64, 8, (1, 255, 257, 700, 833)),      # (the streaming kernel: runs of one, two and four patches)
    (4, 25, 42, 2048, 512, 1, (1, 257, 2560, 4096)),        # (conv1 of 32 chunks)
]


@pytest.mark.parametrize("N,H,W,C,M,S,counts", CASES, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_every_cut_gives_the_same_bits(N, H, W, C, M, S, counts):
    cfg = synth.BlockConfig("runs", N, H, W, C, M, S, "bf16", 1.0, 55)
    inp = synth.make_block_inputs(cfg)
    d = U.dev_inputs(inp)
    full = torch.empty_like(d["x"])
    B.lasnet_sparse_bottleneck(d["x"], None, None, S, *U.weights(d), out=full, flags=B.LASNET_FORCE_FUSED)
    few = [0, N - 1]
    f = inp.f64
    ref = O.dense_bottleneck(f["x"][few], f["W1"], f["b1"], f["W2"], f["b2"], f["W3"], f["b3"])
    U.assert_block_close(full[few], ref, d["x"][few], np.ones((len(few), H, W)), "bf16", "full")
    want, untouched = U.bits(full), U.bits(torch.tensor(777.0, dtype=torch.bfloat16))
    packed = B.lasnet_pack_weights(S, d["W1"], d["W2"], d["W3"])
    rng = np.random.default_rng(5)
    for count in counts:
        for order in ("ascending", "shuffled", "with invalid entries"):
            cells = rng.permutation(cfg.P)[:count].astype(np.int32)
            if order == "ascending":
                cells.sort()
            entries = cells
            if order == "with invalid entries":              # (the last of a run too)
                cells = cells[:count - count // 3]
                entries = rng.permutation(np.concatenate([cells, rng.choice([-1, cfg.P, -(1 << 31), 1 << 30], count // 3)])).astype(np.int32)
            idx, cnt = U.list_tensor(entries, cfg.P), torch.tensor([count], dtype=torch.int32, device="cuda")
            out = torch.full_like(d["x"], 777.0)
            B.lasnet_sparse_bottleneck_packed(d["x"], idx, cnt, S, M, packed, d["b1"], d["b2"], d["b3"], out=out,
                                              flags=B.LASNET_FORCE_FUSED | B.LASNET_SKIP_IDENTITY)
            mask = np.zeros(cfg.P, bool)
            mask[cells] = True
            up = mask.reshape(N, H // S, W // S).repeat(S, 1).repeat(S, 2)
            got = U.bits(out)
            assert np.array_equal(got[up], want[up]), (count, order)
            assert (got[~up] == untouched).all(), (count, order)


@pytest.mark.parametrize("N,H,W,C,M,S,counts", CASES[-2:], ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_counted_waits_against_drained_barriers(monkeypatch, N, H, W, C, M, S, counts):
    """Bit for bit as the build whose barriers wait for everything: runs of several patches (the streaming kernel's windows are requested
    two patches ahead, and what its stores leave in flight is counted), with entries inside them that store nothing; and every
    number of row blocks that conv1 of 32 chunks has."""
    from paper_2210_06223_amd import build
    check = B.load_library(build.LIB_CHECK)
    cfg = synth.BlockConfig("counts", N, H, W, C, M, S, "bf16", 1.0, 56)
    d = U.dev_inputs(synth.make_block_inputs(cfg, want_f64=False))
    packed = B.lasnet_pack_weights(S, d["W1"], d["W2"], d["W3"])
    rng = np.random.default_rng(6)
    lists = [np.sort(rng.permutation(cfg.P)[:n]) for n in counts]
    if C == 2048:                                            # runs of 1 to 16 cells anywhere: 9 to 96 rows
        lists = [rng.permutation(cfg.P)[:256 * n] for n in (1, 2, 3, 4, 5, 7, 9, 10, 11, 16)]
    for cells in lists:
        for invalid in (False, True):
            entries = cells.astype(np.int32)
            if invalid:
                entries[rng.random(len(entries)) < 0.3] = cfg.P
            idx, cnt = U.list_tensor(entries, cfg.P), torch.tensor([len(entries)], dtype=torch.int32, device="cuda")
            outs = []
            for library in (B.lib(), check):
                monkeypatch.setattr(B, "_lib", library)
                out = torch.full_like(d["x"], 777.0)
                B.lasnet_sparse_bottleneck_packed(d["x"], idx, cnt, S, M, packed, d["b1"], d["b2"], d["b3"], out=out,
                                                  flags=B.LASNET_FORCE_FUSED | B.LASNET_SKIP_IDENTITY)
                outs.append(U.bits(out))
                monkeypatch.undo()
            assert np.array_equal(*outs), (len(entries), invalid)
