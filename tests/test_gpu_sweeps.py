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


def _obstacles(nx, ny):
    t = I.channel(nx, ny)
    rng = np.random.default_rng(nx)
    inner = t[2:-2, 3:-3]
    inner[rng.random(inner.shape) < 0.03] = 0
    return t


# Strips are 64 - 2 steps columns wide: the widths leave a last strip of one
# column (151 = 3 * 50 + 1, 157, 169), of less than the halo, and a full one;
# the heights give segments of four rows and up, ragged and shorter than the
# halo, and a lattice of fewer rows than the halo has.
@pytest.mark.parametrize("steps", [1, 2, 4, 6, 7])
@pytest.mark.parametrize("shape", [(128, 6), (151, 37), (157, 66), (169, 130), (200, 70),
                                   (312, 301), (1100, 523)])
@pytest.mark.parametrize("prec", [lbm.LBM_F64, lbm.LBM_F32, lbm.LBM_F32_S_F16, lbm.LBM_F32_S_BF16])
def test_marching_sweep_matches_single_steps(prec, shape, steps, monkeypatch):
    """The marching sweep (several steps in registers, one wave per strip and
    segment) has the bits of one launch per step, over intervals whose last
    launch takes every shorter step count, a run the device stops, an exchange
    step, and the statistics."""
    if prec == lbm.LBM_F64 and steps > 4:
        pytest.skip("the FP64 form marches four steps at most")
    print(f"march {shape} prec={prec} steps={steps}", flush=True)
    t = _obstacles(*shape)
    res = []
    for env in ({"LBM_TB": "0"}, {"LBM_TB": "1", "LBM_MARCH": str(steps)}):
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        g = lbm.Lattice(t, 0.7, 0.04, precision=prec)
        out = [g.run(97, 0.0, 13)[:2], g.state(), g.run(400, 2e-2, 9)[:2], g.state()]
        r = g.run(45, 0.0, 15)[2]
        if shape[1] > 8:
            g.shape_update(frac=0.02, seed=5)
        g.run(31, 0.0, 31)
        out += [g.state(), g.mask(), g.stats()[0], g.bench_sweep(5) > 0, g.state()]
        res.append((out, r))
        g.close()
    for x, y in zip(res[0][0], res[1][0]):
        assert np.array_equal(x, y)
    assert res[1][1] == pytest.approx(res[0][1], rel=1e-12)  # sums grouped differently
