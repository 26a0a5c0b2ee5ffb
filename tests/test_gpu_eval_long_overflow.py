"""Terms of 9 to 16 factors whose partials overflow while shorter products do
not: in complex double every column of them is infinite and none is NaN."""
import numpy as np
import pytest

import paper_1505_00383_amd as ph
from paper_1505_00383_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("k", [9, 10, 11, 13, 15, 16])
def test_overflowing_partials_are_infinite(k):
    n, npts = 16, 70
    s = synth.system_from_terms(n, [[(1.0 + 0j, {v: 1 for v in range(k)})] for _ in range(n)])
    x = np.zeros((npts, n, 2, 1))
    x[:, :, 0, 0] = 10.0 ** (310.0 / (k - 1))  # k - 1 factors: 1e310, k - 2 factors: finite
    S = ph.System(s)
    xs = ph.to_soa(x)
    _, jac = ph.eval_jac(S, xs, npts, 1)
    j = ph.from_soa(jac, npts, (n, n, 2, 1))
    assert np.all(j[:, :, :k, 0] == np.inf) and np.all(j[:, :, :k, 1] == 0)
