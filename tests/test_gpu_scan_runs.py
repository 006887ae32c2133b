"""The scan of the route workgroups' histograms where its runs of rows change: none, one or several rows each, more than one batch
of 16, the last run short or empty; experts that do not fill the last workgroup's 16."""
import pytest

from test_gpu_route_tables import m, test_route_tables as check       # noqa: F401  (m: the fixture)

pytestmark = pytest.mark.gpu


# experts, top-k, tokens, tp, slices: every unit has a route workgroup of its own
@pytest.mark.parametrize("E,k,T,tp,S", [(15, 2, 63, 1, 63), (17, 1, 130, 1, 65), (33, 2, 129, 3, 43), (5, 1, 2048, 4, 256),
                                        (16, 1, 4100, 5, 205), (20, 2, 2176, 1, 1088)])
def test_runs(m, E, k, T, tp, S):                   # noqa: F811
    check(m, E, k, T, tp, S, False)
