"""The slab schedule (a few images of a deep stage) at the edges of its tiles and at both ends of its range."""
import numpy as np
import pytest
import torch

from paper_2210_06223_amd import binding as B
from paper_2210_06223_amd import synth
from tests import _util as U
from tests.test_gpu_parity import _cfg, _run_case

pytestmark = pytest.mark.gpu

CASES = [
    _cfg("stage3_b128", N=1, name="s3_one_image"),
    _cfg("stage3_b128", N=3, S=7, name="s3_S7_ragged"),                                     # 49 rows: a block of one row
    _cfg("stage3_b128", N=1, S=1, name="s3_pixels"),
    synth.BlockConfig("s3_6x10", 2, 6, 10, 1024, 256, 2, "bf16", 0.5, 91),                  # not square
    synth.BlockConfig("s3_one_cell", 1, 2, 2, 1024, 256, 2, "bf16", 1.0, 92),               # four pixels in all
    _cfg("stage4_b128", N=2, name="s4_two_images"),
    synth.BlockConfig("s4_one_pixel", 1, 1, 1, 2048, 512, 1, "bf16", 1.0, 93),
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_slab_edges(cfg):
    _run_case(cfg, k=max(1, int(round(cfg.r * cfg.P))), flags=B.LASNET_POST_RELU)
    _run_case(cfg, k=cfg.P)
    _run_case(cfg, k=0)


@pytest.mark.parametrize("name,N,S", [("stage3_b128", 5, 2), ("stage3_b128", 16, 2), ("stage3_b128", 11, 1), ("stage3_b128", 24, 7),
                                      ("stage3_b128", 32, 7), ("stage4_b128", 7, 1), ("stage4_b128", 17, 1), ("stage4_b128", 40, 1)])
@pytest.mark.parametrize("r", [0.1, 0.6, 1.0])
def test_slab_matches_the_other_schedules(name, N, S, r):
    """Shuffled lists with entries that are no cells of the map, against the fused or tiled kernels.  Both round y1, y2 and
    out to bf16 at the same points, so they differ only where sums in another order round apart: less than if
    every value did by one place, 2^-8 of its size."""
    cfg = _cfg(name, N=N, S=S, name="%s_n%d_s%d" % (name, N, S))
    d = U.dev_inputs(synth.make_block_inputs(cfg, want_f64=False))
    il = synth.make_index_list(cfg.N, cfg.G, cfg.GW, r, seed=N, order="shuffled")
    if r < 1:
        il = np.concatenate([il[:len(il) // 2], [-1, cfg.P, 1 << 30], il[len(il) // 2:]]).astype(np.int32)
    idx, count = U.list_tensor(il, cfg.P), torch.tensor([len(il)], dtype=torch.int32, device="cuda")
    packed = B.lasnet_pack_weights(S, d["W1"], d["W2"], d["W3"])
    outs = []
    for flags in (0, B.LASNET_FORCE_FUSED if name == "stage3_b128" else B.LASNET_FORCE_TILED):
        out = torch.full_like(d["x"], 777.0)
        B.lasnet_sparse_bottleneck_packed(d["x"], idx, count, S, cfg.M, packed, d["b1"], d["b2"], d["b3"], out=out, flags=flags)
        outs.append(out.double())
    assert torch.isfinite(outs[0]).all()
    rel = ((outs[0] - outs[1]).norm() / outs[1].norm()).item()
    assert rel <= 2.0 ** -8, rel


@pytest.mark.parametrize("raw", [False, True], ids=["packed", "raw"])
def test_capture_leaves_the_library_buffer_alone(raw):
    """A graph may be replayed on any stream, beside later calls on the one it was captured on, so the fused kernel is recorded
    whether or not the stream has a buffer that the slab launches fit in.  (Raw weights are repacked into that buffer: there
    it is as large as a call that ran the fused kernel made it, which has to be enough.)"""
    cfg = _cfg("stage3_b128", N=2, name="s3_captured")
    d = U.dev_inputs(synth.make_block_inputs(cfg, want_f64=False))
    il = synth.make_index_list(cfg.N, cfg.G, cfg.GW, 0.5, seed=3)
    idx, count = U.list_tensor(il, cfg.P), torch.tensor([len(il)], dtype=torch.int32, device="cuda")
    packed = B.lasnet_pack_weights(cfg.S, d["W1"], d["W2"], d["W3"])
    side = torch.cuda.Stream()

    def call(out, flags=0):
        if raw:
            B.lasnet_sparse_bottleneck(d["x"], idx, count, cfg.S, *U.weights(d), out=out, flags=flags)
        else:
            B.lasnet_sparse_bottleneck_packed(d["x"], idx, count, cfg.S, cfg.M, packed, d["b1"], d["b2"], d["b3"], out=out, flags=flags)

    want = torch.empty_like(d["x"])
    call(want, B.LASNET_FORCE_FUSED)
    for warm in ((B.LASNET_FORCE_FUSED, 0) if raw else (None, 0)):
        out = torch.empty_like(d["x"])
        torch.cuda.synchronize()
        if warm is not None:
            with torch.cuda.stream(side):
                call(torch.empty_like(d["x"]), warm)
            torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            call(out)
        for _ in range(3):
            out.fill_(777.0)
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(U.bits(out), U.bits(want)), warm
