"""The back-projection's adjoint at the edges of its forms: planes of one to five 64-wide
pieces, columns of one to four 64-voxel pieces and longer (the form without LDS), voxel
steps along z below 2/3 of a beam-frame pixel (likewise), a first voxel off the axis, and
control points in batches.  Gradients <= 1e-4 of max |g| against the FP64 oracle, the bar
of the other gradient tests; each control point's gradients do not depend on the batch."""
import copy

import numpy as np
import pytest
import torch

import oracle
from paper_2512_18863_amd import inputs
from tests.test_gpu_parity import _say, _t

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (nz, lateral field, kernel width, voxel step along z): 2.5 mm beam-frame pixels
CASES = [
    (1, 10.0, 3, 2.5), (63, 70.0, 13, 2.5), (65, 77.5, 3, 2.5), (128, 140.0, 31, 2.5), (130, 150.0, 15, 2.5),
    (200, 230.0, 3, 2.5), (257, 230.0, 3, 2.5), (40, 310.0, 15, 2.5), (50, 40.0, 5, 1.0), (40, 60.0, 5, 4.0),
]


@pytest.mark.parametrize("nz,field,n_taps,sz", CASES, ids=["%d-%g-%d-%g" % c for c in CASES])
def test_backproject_forms(nz, field, n_taps, sz):
    from paper_2512_18863_amd.engine import DoseEngine
    c = inputs.tiny_case(seed=nz + 1, n_cp=4, n_taps=n_taps, shape=(nz, 11, 9), spacing=2.5, field=field, n_leaf=12,
                         leaf_width=2.0 * field / 12)
    c = copy.copy(c)
    c.spacing = (2.5, 2.5, sz)
    c.origin = (c.origin[0], c.origin[1], -0.5 * (nz - 1) * sz + 0.7)
    c.lat_step = c.depth_step = 2.5
    eng = DoseEngine(c)
    _say("back-projection adjoint nz %d sz %g, planes %d x %d x %d" % (nz, sz, eng.Nk, eng.Nu, eng.Nv))
    w = np.random.default_rng(nz).uniform(size=c.shape).astype(np.float32)
    m = oracle.Model(c)
    ref = oracle.backward(m, oracle.density(m), c.gantry, c.leaves, c.jaws, c.mu, w.astype(np.float64))
    args = (_t(c.leaves), _t(c.jaws), _t(c.mu), _t(w))
    got = eng.backward(*args)
    for name, a, r in zip(("leaves", "jaws", "mu"), got, ref):
        e, top = np.abs(a.cpu().numpy() - r).max(), np.abs(r).max()  # (wide fields: no dose at the jaws, top = 0)
        _say("%s: max|dg| = %.2e, max|g| = %.2e" % (name, e, top))
        assert e <= 1e-4 * top, name
    for a, b in zip(got, DoseEngine(c, max_cp_batch=3).backward(*args)):
        assert torch.equal(a, b)
