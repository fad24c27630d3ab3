"""Timed cases of the sparse bottleneck path: what a program that runs LASNet blocks has this library do.

A case is one block on one batch.  Shapes are the four ResNet-101 stages of synth.CONFIGS with the patch sizes
that Sec. 3.2 / 4.2 consider, the paper's own Table 1 block (56x56x256, S=4, r=0.6, batch 1, fp32), larger and
non-square maps as a detector's backbone has them, and generic widths.  The keys of a case:

  dtype      "bf16" | "f32"
  N H W C M  batch, map, block width, mid width
  S          patch side (0: the static block, no patches)
  r          activation ratio the masker is calibrated to (or the list is drawn with)
  structure  "iid": active cells anywhere | "blob": one foreground region per image
  relu       LASNET_POST_RELU
  entry      which public calls make up the pass:
    step       masker_ex(pass_out) + sparse_bottleneck(plain weights, SKIP_IDENTITY): bench.py's step
    packed     masker_ex(pass_out) + sparse_bottleneck_packed: a block of the ResNet-101 body
    planned    masker_ex(pass_out) + sparse_bottleneck_planned(mask handed on, caller's workspace)
    two_calls  masker + sparse_bottleneck, the identity copy inside the block call
    block      sparse_bottleneck_packed alone on a given list (latency against the ratio)
    dense      dense_bottleneck: the static block that the latency ratio is measured against
"""
from __future__ import annotations

import math

import torch

from paper_2210_06223_amd import binding as B
from paper_2210_06223_amd import synth

# (H = W, C, M, patch sizes with a matrix-core kernel) of the ResNet-101 stages
STAGES = {1: (56, 256, 64, (1, 2, 4, 7, 8)), 2: (28, 512, 128, (1, 2, 4, 7)), 3: (14, 1024, 256, (1, 2, 7)), 4: (7, 2048, 512, (1,))}


def _case(dtype, N, H, W, C, M, S, r, entry, structure="iid", relu=False, name=None):
    c = {"dtype": dtype, "N": N, "H": H, "W": W, "C": C, "M": M, "S": S, "r": r, "structure": structure,
         "relu": relu, "entry": entry}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one image, latency: the 14x14 stage holds 22 of the body's 29 sparse blocks
        _case("bf16", 1, 14, 14, 1024, 256, 2, 0.5, "packed", relu=True, name="s3_b1"),
        # the block of the paper's Table 1, in the paper's precision
        _case("f32", 1, 56, 56, 256, 64, 4, 0.6, "two_calls", "blob", name="table1_f32_b1"),
        # bench.py's workload
        _case("bf16", 128, 14, 14, 1024, 256, 2, 0.5, "step", name="s3_b128"),
        # the other stages at batch size, as the ResNet-101 body runs them
        _case("bf16", 64, 56, 56, 256, 64, 8, 0.4, "packed", relu=True, name="s1_b64"),
        _case("bf16", 128, 28, 28, 512, 128, 4, 0.5, "packed", "blob", relu=True, name="s2_b128"),
        _case("bf16", 128, 7, 7, 2048, 512, 1, 0.5, "planned", relu=True, name="s4_b128"),
        # coarse patches at 14x14 (S = 8-4-7-1 over the stages), a serving batch
        _case("bf16", 24, 14, 14, 1024, 256, 7, 0.4, "packed", relu=True, name="s3_S7_b24"),
        # a detector's map: large, not square, few images; a list from elsewhere
        _case("bf16", 2, 100, 168, 512, 128, 4, 0.3, "block", "blob", relu=True, name="s2_100x168_b2"),
        # the static block
        _case("bf16", 128, 14, 14, 1024, 256, 0, 1.0, "dense", name="s3_dense_b128"),
        # fp32 at a deep stage (validation of a trained model against its fp32 weights)
        _case("f32", 16, 14, 14, 1024, 256, 2, 0.5, "step", name="s3_f32_b16"),
        # a width that no ResNet-101 stage has, ragged batch, a map that is not square
        _case("bf16", 13, 28, 20, 192, 48, 4, 0.5, "step", name="c192_b13"),
        # large batch, finer patches at the first stage
        _case("bf16", 256, 56, 56, 256, 64, 4, 0.4, "packed", "blob", relu=True, name="s1_S4_b256"),
    ]


def _fits_generic(M, S):
    """Patches that the shape-generic kernel's LDS holds."""
    return ((S + 2) ** 2 + S * S) * M * 4 <= 159 * 1024


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def draw(rng):
    cases = {c["name"]: c for c in listed()}
    kind = rng.choices(("stage", "map", "f32", "width"), (11, 3, 3, 3))[0]
    r = round(rng.uniform(0.1, 1.0), 3)
    structure = rng.choice(("iid", "blob"))
    relu = rng.random() < 0.5
    if kind in ("stage", "map"):
        H, C, M, sizes = STAGES[rng.choice((1, 2, 3, 4))]
        S = rng.choice(sizes)
        W = H
        entry = rng.choice(("step", "packed", "packed", "planned", "two_calls", "block", "dense"))
        N = _log_int(rng, 1, 256)
        if kind == "map":                       # about 800 x 1333 pixels at this stage, in whole patches
            H, W = (max(1, int(v * H / 56 * rng.uniform(0.5, 1.0)) // S) * S for v in (200, 336))
            N = rng.randint(1, 4)
        limit, dtype = _cost(cases["s1_S4_b256"]), "bf16"
    elif kind == "f32":
        H, C, M, sizes = STAGES[rng.choice((1, 2, 3, 4))]
        S = rng.choice([s for s in sizes if _fits_generic(M, s)])
        W, N = H, _log_int(rng, 1, 16)
        entry = rng.choice(("step", "two_calls", "dense"))
        limit, dtype = _cost(cases["s3_f32_b16"]), "f32"
    else:
        M = 4 * rng.randint(3, 40)
        C = 4 * M
        S = rng.choice([s for s in (1, 2, 3, 4, 5, 7) if _fits_generic(M, s)])
        H, W = S * rng.randint(1, max(1, 40 // S)), S * rng.randint(1, max(1, 40 // S))
        N = _log_int(rng, 1, 64)
        entry = rng.choice(("step", "two_calls"))
        limit, dtype = _cost(cases["s3_f32_b16"]) / 4, rng.choice(("bf16", "f32"))
    if entry == "dense":
        S, r = 0, 1.0
    case = _case(dtype, N, H, W, C, M, S, r, entry, structure, relu)
    while _cost(case) > limit and case["N"] > 1:
        case["N"] = case["N"] * 3 // 4
    return case


def _active(case):
    """Share of the pixels that are active, and of those whose conv1 output some active pixel needs."""
    r, S = case["r"], case["S"]
    if case["entry"] == "dense" or case["structure"] == "blob":
        return r, r
    if S == 1:
        return r, 1 - (1 - r) ** 9
    inner, corner = (S - 2) ** 2 / S ** 2, 4 / S ** 2
    edge = 1 - inner - corner
    return r, inner * r + edge * (1 - (1 - r) ** 2) + corner * (1 - (1 - r) ** 4)


def work(case):
    N, H, W, C, M = (case[k] for k in "NHWCM")
    es = 2 if case["dtype"] == "bf16" else 4
    px = N * H * W
    act, need = _active(case)
    weights = (2 * C * M + 9 * M * M) * es + (2 * M + C) * 4
    if case["entry"] == "block":                # the list's pixels and their neighbours in, the list's pixels out
        feature = px * C * es * (need + act)
    else:                                       # the whole map in (masker, or all active), the whole map out
        feature = 2 * px * C * es
    cells = px // max(1, case["S"] ** 2)
    lists = cells * (1 + 4 * act) if case["entry"] not in ("dense", "block") else 4 * cells * act if case["S"] else 0
    return {"bytes": feature + weights + lists,
            "flops": px * (need * 2 * C * M + act * (18 * M * M + 2 * C * M))}


def tolerance(case):
    # Against the same block in fp64 (masks and lists as they are): fp32 results are off by up to rel 5e-7, max 4e-6;
    # bf16 ones, with y1 and y2 rounded to bf16, by rel 2.8e-3, max 2.1e-2; and where no matrix-core kernel exists the
    # block keeps y1 and y2 in fp32 and only its last rounding shows, rel 2e-5, max 7e-3.  Four times that.  Masks, lists
    # and counts are the same whole numbers in every correct implementation (their margin to the threshold is far
    # above what fp64 sums differ by).
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 1.6e-5, "differ": 0.0}
    if (case["C"], case["M"]) in [s[1:3] for s in STAGES.values()]:
        return {"rel": 1.1e-2, "max": 8e-2, "differ": 0.0}
    return {"rel": 8e-5, "max": 3e-2, "differ": 0.0}


def _foreground(N, H, W, g, dev):
    """[N,H,W]: a smooth bump around a random centre of each image, 1 at the centre."""
    cy, cx = torch.rand((2, N, 1, 1), generator=g, device=dev)
    yy = (torch.arange(H, device=dev) + 0.5).view(1, H, 1) / H
    xx = (torch.arange(W, device=dev) + 0.5).view(1, 1, W) / W
    return torch.exp(-((yy - cy) ** 2 + (xx - cx) ** 2) / 0.18)


def prepare(case, seed):
    dev = torch.device("cuda")
    N, H, W, C, M, S = (case[k] for k in "NHWCMS")
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device=dev).manual_seed(seed)

    def normal(*shape, std=1.0, mean=0.0):
        return torch.randn(shape, generator=g, device=dev) * std + mean

    # He-normal weights with the batch norm's scale folded in, small biases
    st = {"case": case, "S": S, "M": M,
          "W1": (normal(M, C, std=math.sqrt(2 / C)) * normal(M, 1, std=0.1, mean=1.0)).to(dt),
          "W2": (normal(M, 3, 3, M, std=math.sqrt(2 / (9 * M))) * normal(M, 1, 1, 1, std=0.1, mean=1.0)).to(dt),
          "W3": (normal(C, M, std=math.sqrt(2 / M)) * normal(C, 1, std=0.1, mean=1.0)).to(dt),
          "b1": normal(M, std=0.1), "b2": normal(M, std=0.1), "b3": normal(C, std=0.1)}
    Wm = st["Wm"] = normal(C, std=0.02)
    masked = case["entry"] not in ("dense", "block")

    # block inputs follow a ReLU; a foreground region answers the masker's weights
    x = st["x"] = torch.empty((N, H, W, C), dtype=dt, device=dev)
    fg = _foreground(N, H, W, g, dev) if masked and case["structure"] == "blob" else None
    score = torch.empty((N, H, W), dtype=torch.float64, device=dev)
    step = max(1, (64 << 20) // (H * W * C))
    for n in range(0, N, step):
        v = normal(min(step, N - n), H, W, C)
        if fg is not None:
            v += fg[n:n + step, :, :, None] * torch.sign(Wm)
        x[n:n + step] = torch.relu_(v).to(dt)
        if masked:
            score[n:n + step] = (x[n:n + step].float() @ Wm).double()
        del v
    st["out"] = torch.empty_like(x)
    st["flags"] = B.LASNET_POST_RELU if case["relu"] else 0
    if case["entry"] == "dense":
        return st

    G, GW = H // S, W // S
    P = N * G * GW
    st["mask"] = torch.zeros((N, G, GW), dtype=torch.uint8, device=dev)
    st["idx"] = torch.zeros((P,), dtype=torch.int32, device=dev)
    st["count"] = torch.zeros((1,), dtype=torch.int32, device=dev)
    if masked:
        # the masker's bias: the threshold lies midway between two neighbouring logits
        logit = score.view(N, G, S, GW, S).mean(dim=(2, 4)).flatten().sort(descending=True).values
        k = min(P, max(1, round(case["r"] * P)))
        edge = logit[k - 1] - 1.0 if k == P else 0.5 * (logit[k - 1] + logit[k])
        st["bm"] = -float(edge)
    else:
        ids = synth.make_index_list(N, G, GW, case["r"], seed=seed, structure=case["structure"])
        st["idx"][:len(ids)] = torch.from_numpy(ids).to(dev)
        st["count"].fill_(len(ids))
        st["out"].copy_(x)                      # the caller's pass-through: SKIP_IDENTITY
    if case["entry"] in ("packed", "planned", "block"):
        st["packed"] = B.lasnet_pack_weights(S, st["W1"], st["W2"], st["W3"])
    if case["entry"] == "planned":
        nbytes = B.lasnet_workspace_bytes(x, M, S)
        st["workspace"] = torch.empty((nbytes,), dtype=torch.uint8, device=dev) if nbytes else None
    return st


def run(st):
    entry, S, x, out, flags = st["case"]["entry"], st["S"], st["x"], st["out"], st["flags"]
    weights = (st["W1"], st["b1"], st["W2"], st["b2"], st["W3"], st["b3"])
    biases = (st["b1"], st["b2"], st["b3"])
    if entry == "dense":
        return B.lasnet_dense_bottleneck(x, *weights, out=out, flags=flags)
    mask, idx, count = st["mask"], st["idx"], st["count"]
    if entry == "two_calls":
        B.lasnet_masker(x, st["Wm"], st["bm"], S, 0.0, mask=mask, idx=idx, count=count)
        B.lasnet_sparse_bottleneck(x, idx, count, S, *weights, out=out, flags=flags)
        return out, mask, idx, count
    flags |= B.LASNET_SKIP_IDENTITY
    if entry == "block":
        return B.lasnet_sparse_bottleneck_packed(x, idx, count, S, st["M"], st["packed"], *biases, out=out, flags=flags)
    B.lasnet_masker_ex(x, st["Wm"], st["bm"], S, 0.0, mask=mask, idx=idx, count=count, pass_out=out)
    if entry == "step":
        B.lasnet_sparse_bottleneck(x, idx, count, S, *weights, out=out, flags=flags)
    elif entry == "packed":
        B.lasnet_sparse_bottleneck_packed(x, idx, count, S, st["M"], st["packed"], *biases, out=out, flags=flags)
    else:
        B.lasnet_sparse_bottleneck_planned(x, idx, count, mask, S, st["M"], st["packed"], *biases, out, st["workspace"],
                                           flags=flags)
    return out, mask, idx, count
