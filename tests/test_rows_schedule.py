"""The row schedule (fp32, and bf16 at widths without a kernel of their own) at the sizes where it can go wrong: 16-row
blocks, groups of 32 channels, 32-deep k-steps, each with remainders; element-wise loads; both ways its waves
share the work; a batch cut into chunks of images; a captured stream, where it may not allocate."""
import numpy as np
import pytest
import torch

from paper_2210_06223_amd import binding as B
from paper_2210_06223_amd import synth
from tests import _util as U
from tests.test_gpu_parity import _run_case

pytestmark = pytest.mark.gpu

CASES = [
    synth.BlockConfig("c1_m1_s1_f32", 1, 1, 1, 1, 1, 1, "f32", 1.0, 61),               # one pixel, one channel
    synth.BlockConfig("c33_m7_s3_bf16", 2, 6, 3, 33, 7, 3, "bf16", 0.5, 62),           # odd width: element-wise loads
    synth.BlockConfig("c36_m20_s2_f32", 3, 6, 10, 36, 20, 2, "f32", 0.4, 63),          # 16-byte pieces, ragged k-step
    synth.BlockConfig("c40_m33_s4_bf16", 2, 8, 12, 40, 33, 4, "bf16", 0.5, 64),        # a second group of one channel
    synth.BlockConfig("c64_m32_s1_f32", 2, 9, 7, 64, 32, 1, "f32", 0.2, 65),           # whole steps and groups
    synth.BlockConfig("c264_m96_s5_bf16", 1, 15, 20, 264, 96, 5, "bf16", 0.6, 66),     # reduction over four waves
    synth.BlockConfig("c64_m16_s8_f32", 6, 40, 40, 64, 16, 8, "f32", 0.5, 67),         # many row tiles; patches of 64 pixels
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_row_schedule_edges(cfg):
    assert B.lasnet_has_fast_path(torch.bfloat16 if cfg.dtype == "bf16" else torch.float32, cfg.C, cfg.M, cfg.S) == 0
    _run_case(cfg, k=int(round(cfg.r * cfg.P)))
    _run_case(cfg, k=cfg.P, flags=B.LASNET_POST_RELU)
    _run_case(cfg, k=0)


def _call(x, idx, count, S, w, flags=0):
    out = torch.full_like(x, 777.0)
    B.lasnet_sparse_bottleneck(x, idx, count, S, *w, out=out, flags=flags)
    return out


def test_chunks_of_images_match_single_images():
    """224x224 pixels of y1 and y2 at M = 256 are 154 MB, so three images run as three chunks: the same launches as
    one image by itself, hence the same bits, with a list that is shuffled over the images."""
    cfg = synth.BlockConfig("chunked", 3, 224, 224, 16, 256, 4, "bf16", 0.3, 71)
    d = U.dev_inputs(synth.make_block_inputs(cfg, want_f64=False))
    w = U.weights(d)
    il = synth.make_index_list(cfg.N, cfg.G, cfg.GW, cfg.r, seed=5, order="shuffled")
    cells = cfg.G * cfg.GW
    got = _call(d["x"], U.list_tensor(il, cfg.P), torch.tensor([len(il)], dtype=torch.int32, device="cuda"), cfg.S, w)
    for n in range(cfg.N):
        one = np.sort(il[il // cells == n]) - n * cells
        want = _call(d["x"][n:n + 1].contiguous(), U.list_tensor(one, cells),
                     torch.tensor([len(one)], dtype=torch.int32, device="cuda"), cfg.S, w)
        assert np.array_equal(U.bits(got[n:n + 1]), U.bits(want)), n


@pytest.mark.parametrize("warm", [False, True])
def test_capture_uses_no_workspace(warm):
    """Under capture nothing is allocated, and a buffer that the stream has is left to its later calls: the one-kernel path is
    recorded instead (its fp32 sums run in another order, K <= 9 * 24 terms of 6e-8 each), which is the noalloc entry's."""
    cfg = synth.BlockConfig("captured", 2, 8, 8, 48, 24, 4, "f32", 0.5, 72)
    d = U.dev_inputs(synth.make_block_inputs(cfg, want_f64=False))
    w = U.weights(d)
    il = synth.make_index_list(cfg.N, cfg.G, cfg.GW, cfg.r, seed=6)
    idx, count = U.list_tensor(il, cfg.P), torch.tensor([len(il)], dtype=torch.int32, device="cuda")
    want = _call(d["x"], idx, count, cfg.S, w)
    out = torch.empty_like(d["x"])
    same = B.lasnet_sparse_bottleneck_noalloc(d["x"], idx, count, cfg.S, *w, out=torch.empty_like(d["x"]))
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    if warm:
        with torch.cuda.stream(side):
            B.lasnet_sparse_bottleneck(d["x"], idx, count, cfg.S, *w, out=out)
        torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        B.lasnet_sparse_bottleneck(d["x"], idx, count, cfg.S, *w, out=out)
    for _ in range(3):
        out.fill_(777.0)
        graph.replay()
        torch.cuda.synchronize()
        err = (out - want).abs().max().item()
        assert err <= 2e-5 * want.abs().max().item(), err
        assert np.array_equal(U.bits(out), U.bits(same))
