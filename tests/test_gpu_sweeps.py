"""Edges of the sweep kernels' own branches, against the oracle or the
general path.  Parity over whole workloads is in the other GPU tests."""
import numpy as np
import pytest

import oracle
from paper_1303_0107_amd import inputs as I
from paper_1303_0107_amd import lbm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    lbm.load()


@pytest.mark.parametrize("exponent", [-560, -513, -512, -511, -300, 0, 300, 510, 511, 512, 560])
def test_f64_quotients_far_from_unit_density(exponent):
    """The FP64 relaxation takes u = j / rho by a shared reciprocal where rho
    lies within 2^+-512 and by division elsewhere.  In a closed box a state
    scaled by 2^n stays scaled by 2^n exactly: states on both sides of both
    limits have the oracle's bits."""
    t = np.zeros((21, 75), np.uint8)
    t[1:-1, 1:-1] = I.FLUID
    rng = np.random.default_rng(7)
    o = oracle.Lattice(t, 0.7, 0.02)
    g = lbm.Lattice(t, 0.7, 0.02)
    f = o.fs * (1.0 + 0.1 * rng.uniform(-1.0, 1.0, o.fs.shape)) * 2.0 ** exponent
    o.fs[:] = f
    g.set_state(f)
    o.run(23, 0.0, 23)
    g.run(23, 0.0, 23)
    live = t != 0
    assert np.isfinite(o.fs[:, live]).all()
    assert np.array_equal(g.state()[:, live], o.fs[:, live])
    g.close()
