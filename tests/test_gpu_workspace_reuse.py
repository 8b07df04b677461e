"""A workspace sized for a larger selection serves a smaller one on the same
matrix, also where only the smaller one's full layout keeps the history of
omega and so asks for more."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import colstore32, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("target", ["self", "explicit"])
def test_workspace_of_a_larger_selection(gpu, target):
    m, n, k = 64, 1 << 18, 16
    A32 = dev(colstore32(synth.planted_dense(m, n, k, 1.3, seed=7)[0]))
    r = 0 if target == "self" else 20
    B = dev(colstore32(np.random.default_rng(8).standard_normal((m, r)))) if r else None
    kw = dict(r_max=r, self_target=r == 0)
    sizes = [gpu.workspace_size(gpu.make_desc(m, n, m, gpu.F32, A32.data_ptr(), None, x, r, r == 0, 0.0, None))
             for x in (k, k + 1)]
    assert sizes[1] < sizes[0]
    res = []
    for ws in (None, torch.empty(sizes[1], dtype=torch.uint8, device="cuda")):
        s = gpu.Selector(A32, m, k_max=k, workspace=ws, **kw)
        s.set_target(B)
        res.append(s.select(k))
        err = s.reconstruction_error(res[-1][0][::-1].copy())
        assert abs(err - res[-1][1][k]) <= 1e-5 * res[-1][1][0]
        s.close()
    assert res[0][2] == res[1][2] == k
    np.testing.assert_array_equal(res[0][0], res[1][0])
    assert np.max(np.abs(res[0][1] - res[1][1])) <= 1e-12 * res[0][1][0]


def test_too_small_a_workspace_is_refused(gpu):
    m, n = 64, 4096
    A = torch.zeros(n, m, device="cuda")
    d = gpu.make_desc(m, n, m, gpu.F32, A.data_ptr(), None, 4, 4, False, 0.0, None)
    ws = torch.empty(gpu.workspace_size(d), dtype=torch.uint8, device="cuda")
    with pytest.raises(gpu.GcssError) as e:
        gpu.create(d, ws.data_ptr(), 1 << 16)
    assert e.value.status == gpu.ERR_WORKSPACE
    with pytest.raises(ValueError):
        gpu.Selector(A, m, k_max=4, r_max=4, workspace=ws[:1 << 16])
