"""The shape-generic scalar kernel against the oracle: it runs where the row schedule may have no workspace (the noalloc entry,
under capture) or is the slower one, and the entry that the other tests go by reaches it for the smallest shapes only."""
import pytest

from paper_2210_06223_amd import binding as B
from tests import _fake_hip as H
from tests import test_gpu_parity as P

CASES = P.GENERIC_CASES + [P._cfg("tiny_f32"), P.synth.BlockConfig("scalar_c33_m7_bf16", 2, 6, 3, 33, 7, 3, "bf16", 0.5, 141),
                           P.synth.BlockConfig("scalar_c64_m48_f32", 3, 9, 7, 64, 48, 1, "f32", 0.4, 142),
                           P.synth.BlockConfig("scalar_c40_m33_bf16", 2, 16, 8, 40, 33, 8, "bf16", 0.6, 143)]


def test_the_noalloc_entry_runs_the_scalar_kernel():
    """(Host only.)  And so does a captured call of the other entry."""
    got = H.run("result = [kernels(call(e, {'f32': F32, 'bf16': BF16}[d], *a, flags=4, capturing=c)[1])[-1] for d, a in %r for e, c in (('noalloc', 0), ('ex', 1))]"
                % [(c.dtype, (c.N, c.H, c.W, c.C, c.M, c.S)) for c in CASES])
    assert {H.kernel_name(n) for n in got} == {"bneck_generic_kernel"}


@pytest.fixture
def noalloc(monkeypatch):
    monkeypatch.setattr(B, "lasnet_sparse_bottleneck", B.lasnet_sparse_bottleneck_noalloc)


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_scalar_kernel_matches_the_oracle(cfg, noalloc):
    P._run_case(cfg, k=int(round(cfg.r * cfg.P)))
    P._run_case(cfg, k=cfg.P, flags=B.LASNET_POST_RELU)
    P._run_case(cfg, k=0)


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,k", [(P._cfg("stage3_b128", N=1, name="scalar_s3"), 25), (P._cfg("stage1_b64", N=1, S=4, name="scalar_s1"), 30)],
                         ids=lambda v: getattr(v, "name", str(v)))
def test_scalar_kernel_on_stage_shapes(cfg, k, noalloc):
    P._run_case(cfg, k=k, flags=B.LASNET_FORCE_GENERIC)


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", [P._cfg("tiny_f32"), P.synth.BlockConfig("scalar_hyg_bf16", 2, 12, 12, 24, 20, 2, "bf16", 0.5, 144)], ids=lambda c: c.name)
def test_scalar_kernel_ignores_what_is_no_cell(cfg, noalloc):
    P.test_count_beyond_capacity_and_invalid_entries(cfg)
