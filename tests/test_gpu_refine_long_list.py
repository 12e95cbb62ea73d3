"""IMPORT lists on either side of the length from which the filter reads a node's
neighbours plane by plane (65536 nodes), against the refined oracle: a flat box
whose shell holds most of its nodes."""
import numpy as np
import pytest

from tests.pair import normwise
from tests.test_gpu_refine import F64_TOL, run_refined

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,longer", [(179, False), (180, True)])
def test_import_list_length_f64(n, longer):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    side = (n, n, 6)
    nodes = np.prod([a - 1 for a in side]) - np.prod([a - 3 for a in side])
    assert (nodes >= 65536) == longer and abs(nodes - 65536) < 1000
    case = dict(name="long-list", q=19, shape=(n + 9, n + 9, 15), lo=(4, 4, 4),
                hi=(n + 4, n + 4, 10), tau=0.55)
    g0, g1, og, _, _ = run_refined(case, 2)
    skip = og.crole == 2  # COVERED coarse nodes are never updated
    assert normwise(g0[:, ~skip], og.coarse.f[:, ~skip]) <= F64_TOL
    assert normwise(g1, og.fine.f) <= F64_TOL
