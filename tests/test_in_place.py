"""The in-place update on either schedule that allows it, at the 7x7 stage."""
import pytest

from paper_2210_06223_amd import binding as B
from tests import _fake_hip as H
from tests import test_gpu_parity as P


def test_what_an_in_place_call_runs():
    """(Host only.)  A few images the slab schedule, more of them or on request the tiled one; 14x14x1024 only on request."""
    got = H.run("""
result = [[st, kernels(ev)] for st, ev in (call('packed', BF16, *a, flags=f, in_place=True) for a, f in
          (((5, 7, 7, 2048, 512, 1), 0), ((5, 7, 7, 2048, 512, 1), 16), ((41, 7, 7, 2048, 512, 1), 0), ((4, 14, 14, 1024, 256, 2), 0)))]
""")
    names = ["+".join(sorted({H.kernel_name(k).split("_")[0] for k in ks})) for _, ks in got]
    assert [st for st, _ in got] == [0, 0, 0, B.LASNET_EALIAS] and names == ["slab", "tiled", "tiled", ""]


@pytest.mark.gpu
def test_in_place_on_the_tiled_kernels_of_the_7x7_stage():
    P.test_in_place_update_on_the_tiled_schedule(P._cfg("stage4_b128", N=5, name="s4_inplace_tiled"), B.LASNET_FORCE_TILED)
