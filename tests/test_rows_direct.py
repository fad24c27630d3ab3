"""Row-schedule calls with few cells: the copy as a part of the first launch, and the convolutions on the caller's own weights
with no plan, at the edges of their ranges; and both against the plan's launches, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2210_06223_amd import binding as B
from paper_2210_06223_amd import synth
from tests import _fake_hip as H
from tests import _util as U
from tests.test_gpu_parity import _run_case

# (N, H, W, C, M, S) -> whether the copy rides, whether there is no plan
ROUTES = [
    ((8, 8, 8, 64, 32, 1), True, True),                  # 512 cells
    ((3, 9, 19, 64, 32, 1), False, False),               # 513
    ((1, 56, 56, 256, 64, 4), True, False),              # fp32: too many fragments for the natural layout
    ((2, 12, 20, 40, 24, 4), True, True),                # ragged k-steps and groups
    ((1, 20, 20, 320, 88, 2), True, True),               # three groups of channels
    ((2, 14, 14, 128, 104, 7), True, False),             # four
    ((3, 21, 14, 68, 36, 7), True, True),                # bf16 cannot read 16-byte pieces of it: its copy and plan as ever
]

# (dtype, shape) -> whether there is no plan: both sides of each line of direct_is_faster
EDGES = [
    ("f32", (11, 32, 32, 128, 32, 8), True),             # 12.0 thousand fragments, four k-steps
    ("f32", (5, 28, 28, 192, 48, 4), False),             # 14.7 thousand, six
    ("f32", (1, 28, 28, 320, 80, 4), True),              # 6.9 thousand, ten
    ("f32", (1, 28, 28, 352, 88, 4), False),             # 7.2 thousand, eleven
    ("f32", (1, 8, 8, 384, 96, 4), False),               # twelve
    ("bf16", (32, 32, 32, 128, 32, 8), True),            # 34.8 thousand, four
    ("bf16", (10, 28, 35, 192, 48, 7), False),           # 36.8 thousand, six
    ("bf16", (4, 32, 32, 224, 56, 4), True),             # 16.4 thousand, seven
    ("bf16", (8, 32, 32, 224, 56, 8), False),            # 32.8 thousand, seven
]


@pytest.mark.parametrize("dtype,shape,direct", EDGES)
def test_where_the_plan_begins(dtype, shape, direct):
    """(Host only.)"""
    names = H.run("result = kernels(call('ex', %s, *%r)[1])" % ("F32" if dtype == "f32" else "BF16", shape))
    names = [H.kernel_name(n).split("<")[0] for n in names]
    assert names == ([] if direct else ["rows_plan_kernel"]) + ["rows_conv%d_kernel" % k for k in (1, 2, 3)], names


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,shape,direct", EDGES)
def test_either_side_of_the_line(dtype, shape, direct):
    cfg = synth.BlockConfig("direct", *shape, dtype, 0.4, 137)
    _run_case(cfg, k=max(1, int(round(cfg.r * cfg.P))))


def test_routes():
    """(Host only.)"""
    got = H.run("result = [[kernels(call('ex', d, *a, flags=f)[1]) for f in (0, 4)] for a in %r for d in (F32, BF16)]" % [r[0] for r in ROUTES])
    for i, (shape, rides, direct) in enumerate(ROUTES):
        for j, dtype in enumerate(("f32", "bf16")):
            if dtype == "bf16" and shape[3:] == (256, 64, 4):
                continue                                 # (a matrix-core kernel of its own)
            pieces = dtype == "f32" or shape[3] % 8 == 0
            convs = ["rows_conv%d_kernel" % k for k in (1, 2, 3)]
            plan = [] if direct and pieces and (dtype == "f32" or shape[4] % 8 == 0) else ["rows_plan_kernel"]
            names = [[H.kernel_name(n).split("<")[0] for n in c] for c in got[2 * i + j]]
            assert names[0] == ([] if rides and pieces else ["copy_kernel"]) + plan + convs, (shape, dtype, names[0])
            assert names[1] == plan + convs, (shape, dtype, names[1])


def test_workgroups_of_the_copy():
    """(Host only.)  Four pieces of 16 bytes per thread, up to 1024 workgroups, whichever launch the copy is a part of."""
    maps = [((1, 8, 8, 64, 32, 1), 1), ((1, 56, 56, 256, 64, 4), 196), ((32, 14, 14, 1024, 256, 7), 1024),
            ((128, 14, 14, 2048, 64, 7), 1024), ((32, 112, 112, 96, 24, 28), 1024)]
    got = H.run("result = [[[int(e[2]) for e in call('ex', F32, *a, flags=f)[1] if e[0] == 'launch'] for f in (0, 4)] for a in %r]" % [m[0] for m in maps])
    for (shape, copy), (with_copy, without) in zip(maps, got):
        assert [a - b for a, b in zip(with_copy, without)] == [copy] + [0] * (len(without) - 1), (shape, with_copy, without)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [r[0] for r in ROUTES], ids=lambda s: "x".join(map(str, s)))
def test_few_cells(shape, dtype):
    cfg = synth.BlockConfig("direct", *shape, dtype, 0.4, 131)
    _run_case(cfg, k=max(1, int(round(cfg.r * cfg.P))))
    _run_case(cfg, k=cfg.P, flags=B.LASNET_POST_RELU)
    _run_case(cfg, k=0)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [ROUTES[0][0], ROUTES[3][0], ROUTES[4][0]], ids=lambda s: "x".join(map(str, s)))
def test_same_bits_as_with_a_plan(shape, dtype):
    """Weights that are not 16-byte aligned have a plan; the sums run in the same order.  Shuffled lists with entries that are no cells,
    counts beyond the list and none, on a workspace that an earlier call has filled with other values."""
    cfg = synth.BlockConfig("direct", *shape, dtype, 0.4, 132)
    d = U.dev_inputs(synth.make_block_inputs(cfg, want_f64=False))
    w = list(U.weights(d))
    moved = torch.empty(w[0].numel() + 1, dtype=w[0].dtype, device="cuda")[1:].view(w[0].shape)
    moved.copy_(w[0])
    other = [t + 1 for t in w]
    rng = np.random.default_rng(9)
    for n, count in ((0, 0), (1, 1), (cfg.P // 3, cfg.P // 3), (cfg.P, cfg.P), (cfg.P, cfg.P + 7), (cfg.P, -5)):
        il = rng.permutation(cfg.P)[:n].astype(np.int32)
        if n > 4:
            il[::5] = rng.choice([-1, cfg.P, -(1 << 31), 1 << 30], len(il[::5]))
        idx, cnt = U.list_tensor(il, cfg.P), torch.tensor([count], dtype=torch.int32, device="cuda")
        outs = []
        for W1 in (w[0], moved):
            B.lasnet_sparse_bottleneck(d["x"] + 1, None, None, cfg.S, *other, out=torch.empty_like(d["x"]))
            out = torch.full_like(d["x"], 777.0)
            B.lasnet_sparse_bottleneck(d["x"], idx, cnt, cfg.S, W1, *w[1:], out=out)
            outs.append(U.bits(out))
        assert np.array_equal(*outs), (n, count)
    outs = [U.bits(B.lasnet_sparse_bottleneck(d["x"], None, None, cfg.S, W1, *w[1:], out=torch.empty_like(d["x"]))) for W1 in (w[0], moved)]
    assert np.array_equal(*outs)
