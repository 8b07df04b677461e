"""The parts of the workspace that only make calls faster do not push a problem
out of the static entry point's array: B = A problems that fit it without them
by a margin of a few percent."""
import pytest

import paper_1312_6838_amd as g


@pytest.mark.parametrize("m,n,k,r", [(256, 62000, 50, 0), (512, 13000, 500, 0), (512, 15000, 200, 64)])
def test_gram_problem_near_the_static_limit_stays_in(m, n, k, r):
    d = g.make_desc(m, n, m, g.F32, 1 << 20, None, k, r, True, 0.0, None)
    assert 0.8 * g.STATIC_SCRATCH_BYTES < g.workspace_size(d) <= g.STATIC_SCRATCH_BYTES
