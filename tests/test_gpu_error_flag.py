"""An error flag raised by the sort kernels ends the call, also where the
layers themselves were made without a sort and are sorted to be read back."""

import pytest

pytestmark = pytest.mark.gpu

from paper_2509_19162_amd import _native as N  # noqa: E402
from paper_2509_19162_amd import api  # noqa: E402
from paper_2509_19162_amd import inputs as I  # noqa: E402


@pytest.mark.parametrize("n,fam,kw", [(10, "pancake", {}), (13, "lrx", {"max_frontier": 100_000}),
                                      (13, "lrx", {"max_frontier": 100_000, "packed_sort": True})])
def test_a_failed_sort_is_reported(n, fam, kw):
    gens = I.family(fam, n)
    eng = api.Engine()
    kw = dict(kw, export_layers=2_000_000)
    eng.run(n, gens, **kw)
    assert N.lib().cg_test_raise_error_flag(eng._e) == N.CG_OK
    with pytest.raises(api.CGError) as e:
        eng.run(n, gens, **kw)
    assert e.value.code == N.CG_E_DEVICE
    eng.close()
