"""The gradient of a batch whose graphs fit a launch each but not one together
(2^24 workgroups of 256 threads are 2^32 threads, which a launch does not
take): edgeless graphs, whose MIS gradient is 1 everywhere."""
import types

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("rows", [(33554432, 33554432, 9), (2 ** 25 - 4, 2 ** 25, 1), (5, 2 ** 26 - 20, 2 ** 23)])
def test_gradient_of_more_rows_than_a_launch(rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2605_06921_amd import mqo
    n, B = sum(rows), 33  # 64 lanes a row, 4 rows a workgroup
    g = types.SimpleNamespace(n=n, row_ptr=np.zeros(n + 1, np.int32), col_idx=np.zeros(0, np.int32), weight=None,
                              vtx_offset=np.concatenate([[0], np.cumsum(rows)]).astype(np.int64))
    dg = mqo.DeviceGraph(g, DEV)
    X = torch.full((n, B), 0.25, device=DEV)
    _, grad = mqo.objective_grad("mis", dg, X, 2.0, want_f=False)
    assert int((grad != 1.0).sum()) == 0
    del X, grad
    torch.cuda.empty_cache()
