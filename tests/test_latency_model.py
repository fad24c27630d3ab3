"""The latency predictor (Sec. 3.3 / App. A re-parameterised for this library on MI355X): its replay of
the kernels' work split, and its predictions against the measured sweeps stored under profiles/."""
import os

import numpy as np

from paper_2210_06223_amd import latency_model as LM
from paper_2210_06223_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_replay_of_the_fused_kernels_work_split():
    cfg = synth.CONFIGS["stage3_b128"]
    idx = np.arange(0, cfg.P, 2, dtype=np.int32)                # 3136 of 6272 cells
    wgs = LM.simulate_fused(idx, cfg.N, cfg.H, cfg.W, cfg.C, cfg.M, cfg.S)
    assert len(wgs) == 256                                      # one round of one workgroup per CU
    assert sum(len(w) for w in wgs) >= 256
    out_blocks = sum(b2 for w in wgs for _, b2 in w)
    assert out_blocks * 16 >= len(idx) * cfg.S * cfg.S          # every active pixel is in some 16-row block
    # isolated cells (no shared window pixels): 16 of them need 16 * 16 rows > 160, so batches are cut
    iso = np.array([n * 49 + gy * 7 + gx for n in range(64) for gy in (0, 2, 4, 6) for gx in (0, 2, 4, 6)], np.int32)
    wgs = LM.simulate_fused(iso, cfg.N, cfg.H, cfg.W, cfg.C, cfg.M, cfg.S)
    assert all(b1 <= 10 for w in wgs for b1, _ in w)            # never more than R1MAX = 160 rows
    # an empty list costs nothing to replay
    assert LM.simulate_fused(np.zeros(0, np.int32), cfg.N, cfg.H, cfg.W, cfg.C, cfg.M, cfg.S) == []


def test_runs_of_several_rounds_cover_the_list_once():
    """Whatever the remainders, and with no run that needs a second batch."""
    for nact, P, PPW, slots in ((50176, 50176, 4, 512), (20071, 50176, 4, 512), (513, 600, 1, 512), (1025, 1027, 1, 512), (8193, 9000, 16, 512),
                                (6271, 6272, 16, 256), (4099, 6272, 4, 256), (511, 6272, 4, 512), (7, 49, 32, 256), (1, 1, 4, 512)):
        spans = LM.fused_runs(nact, P, PPW, slots)
        assert sorted(i for a, b in spans for i in range(a, b)) == list(range(nact)), (nact, P)
        assert max(b - a for a, b in spans) <= PPW and min(b - a for a, b in spans) >= 1, (nact, P)


def test_runs_are_dealt_to_the_xcds_as_the_kernel_does():
    """The list's first runs are the longer ones; a round's share of them is spread over the 8 XCDs, whose runs are neighbours."""
    for nact, P, PPW, slots in ((50176, 50176, 4, 512), (20071, 50176, 4, 512), (3236, 6272, 32, 256), (1025, 1027, 1, 512), (6271, 6272, 16, 256)):
        spans = LM.fused_runs(nact, P, PPW, slots)
        nt, q = len(spans), nact // len(spans)
        for r0 in range(0, nt, slots):
            part = spans[r0:r0 + slots]
            t0 = nt - r0 - len(part)                               # the round's first run in the list
            longer = min(t0 + len(part), nact - q * nt) - min(t0, nact - q * nt)
            assert part[0][0] == t0 * q + min(t0, nact - q * nt)
            for k in range(8):
                mine = part[k::8]
                n = longer // 8 + (k < longer % 8)
                assert [b - a for a, b in mine] == [q + 1] * n + [q] * (len(mine) - n), (nact, r0, k)
                assert [a for a, _ in mine[1:]] == [b for _, b in mine[:-1]]


def test_short_lists_have_one_run_per_cu():
    for nact, runs in ((1, 1), (255, 255), (300, 256), (640, 256), (641, 512)):
        spans = LM.fused_runs(nact, 2100, 4, 512, 640)
        assert len(spans) == runs and sorted(i for a, b in spans for i in range(a, b)) == list(range(nact)), nact
        assert max(b - a for a, b in spans) <= 4


def test_short_lists_are_predicted_with_their_workgroups_alone():
    """Measured on 2 maps of 100x168x512, S=4, cells anywhere: either side of the line, where the second workgroup of a CU comes in."""
    for nact, us in ((256, 11.2), (512, 13.4), (640, 15.9), (768, 16.0), (769, 17.9), (1024, 19.7), (2000, 35.2)):
        idx = np.sort(np.random.default_rng(0).choice(2100, nact, replace=False))
        assert abs(LM.predict_us(idx, 2, 100, 168, 512, 128, 4, "fused") / us - 1) < 0.15, nact


def test_window_pixels_counts():
    assert len(LM.window_pixels([(0, 0, 0)], 2, 14, 14)) == 9          # corner patch: 3 x 3 in the image
    assert len(LM.window_pixels([(0, 3, 3)], 2, 14, 14)) == 16         # interior: 4 x 4
    assert len(LM.window_pixels([(0, 3, 3), (0, 3, 4)], 2, 14, 14)) == 24   # neighbours share 2 columns


def test_predictions_against_the_stored_sweeps():
    worst = 0.0
    n = 0
    for line in open(os.path.join(ROOT, "profiles", "ratio_sweeps_mi355x.txt")):
        if line.startswith("#") or not line.strip():
            continue
        name, sch, r, structure, active, measured, _ = line.split()
        cfg = synth.CONFIGS[name]
        il = synth.make_index_list(cfg.N, cfg.G, cfg.GW, float(r), seed=cfg.seed, structure=structure)
        assert len(il) == int(active)
        pred = LM.predict_us(il, cfg.N, cfg.H, cfg.W, cfg.C, cfg.M, cfg.S, sch)
        worst = max(worst, abs(pred / float(measured) - 1.0))
        n += 1
    assert n >= 50 and worst < 0.15, worst


def test_predicted_latency_does_not_fall_when_more_is_active():
    cfg = synth.CONFIGS["stage4_b128"]
    prev = 0.0
    for r in (0.1, 0.3, 0.5, 0.8, 1.0):
        il = synth.make_index_list(cfg.N, cfg.G, cfg.GW, r, seed=3, structure="blob")
        t = LM.predict_us(il, cfg.N, cfg.H, cfg.W, cfg.C, cfg.M, cfg.S, "tiled")
        assert t >= prev - 1e-9
        prev = t


def test_slab_predictions_against_the_stored_sweep_and_the_librarys_own_choice():
    """Host side of the library by a recording HIP runtime: the schedule that schedule_of names is the one that runs."""
    from tests import _fake_hip as H
    worst, n = 0.0, 0
    for line in open(os.path.join(ROOT, "profiles", "slab_sweep_mi355x.txt")):
        if line.startswith("#"):
            continue
        v = line.split()
        shape = tuple(map(int, v[:6]))
        il = np.arange(int(v[7]))
        assert LM.schedule_of(*shape) == "slab"
        pred = LM.predict_us(il, *shape, "auto")
        assert abs(pred - float(v[9])) < 0.06
        worst, n = max(worst, abs(pred / float(v[8]) - 1)), n + 1
    assert n > 100 and worst < 0.2, worst
    shapes = [(N, h, w, C, M, S) for C, M, S, hw in ((1024, 256, 1, 14), (1024, 256, 2, 14), (1024, 256, 7, 14), (2048, 512, 1, 7), (512, 128, 4, 28))
              for N in (1, 10, 11, 16, 17, 32, 33, 40, 41, 128) for h, w in ((hw, hw), (hw, 3 * hw))]
    got = H.run("result = [kernels(call('packed', BF16, *a, flags=4)[1])[-1] for a in %r]" % shapes)
    for shape, name in zip(shapes, got):
        assert H.kernel_name(name).split("_")[0] == LM.schedule_of(*shape), shape
