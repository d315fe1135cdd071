"""The back-projection's adjoint on planes of 193 to 256 pixels (four 64-wide pieces) over
columns of one to four 64-voxel pieces, with openings as tall as the field: the upper and
lower jaw and the outer leaves lie in the first and last piece, inside the grid.  Gradients
<= 1e-4 of max |g| against the FP64 oracle, the bar of the other gradient tests, and none
of the parameters compared is without a gradient."""
import copy

import numpy as np
import pytest
import torch

import oracle
from paper_2512_18863_amd import inputs
from tests.test_gpu_parity import _say, _t

pytestmark = pytest.mark.gpu


# (nz, lateral field, kernel width, voxel step along z): 2.5 mm beam-frame pixels
CASES = [(130, 240.0, 3, 4.0), (64, 240.0, 3, 8.0), (202, 250.0, 3, 2.5), (256, 312.0, 5, 2.5), (190, 315.0, 3, 3.4)]


@pytest.mark.parametrize("nz,field,n_taps,sz", CASES, ids=["%d-%g-%d-%g" % c for c in CASES])
def test_four_pieces(nz, field, n_taps, sz):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_18863_amd.engine import DoseEngine
    c = inputs.tiny_case(seed=nz + 1, n_cp=3, n_taps=n_taps, shape=(nz, 11, 9), spacing=2.5, field=field, n_leaf=12,
                         leaf_width=2.0 * field / 12)
    c = copy.copy(c)
    c.spacing = (2.5, 2.5, sz)
    c.origin = (c.origin[0], c.origin[1], -0.5 * (nz - 1) * sz + 0.7)
    c.lat_step = c.depth_step = 2.5
    c.jaws = inputs.jaws_square(3, 9.0, field - 4.0)
    c.leaves = np.stack([np.full((3, 12), -6.3), np.full((3, 12), 5.1)], axis=1)
    c.leaves = c.leaves + np.random.default_rng(nz).uniform(-1.0, 1.0, size=c.leaves.shape)
    eng = DoseEngine(c)
    _say("back-projection adjoint nz %d sz %g, planes %d x %d x %d" % (nz, sz, eng.Nk, eng.Nu, eng.Nv))
    assert 193 <= eng.Nv <= 256
    w = np.random.default_rng(nz).uniform(size=c.shape).astype(np.float32)
    m = oracle.Model(c)
    ref = oracle.backward(m, oracle.density(m), c.gantry, c.leaves, c.jaws, c.mu, w.astype(np.float64))
    args = (_t(c.leaves), _t(c.jaws), _t(c.mu), _t(w))
    got = eng.backward(*args)
    for name, a, r in zip(("leaves", "jaws", "mu"), got, ref):
        r = np.asarray(r)
        far = r if name != "jaws" else r[:, 2:]
        e, top = np.abs(a.cpu().numpy() - r).max(), np.abs(r).max()
        _say("%s: max|dg| = %.2e, max|g| = %.2e, least %.2e" % (name, e, top, np.abs(far).min()))
        assert np.abs(far).min() > 0.0
        assert e <= 1e-4 * top, name
    for a, b in zip(got, DoseEngine(c, max_cp_batch=2).backward(*args)):
        assert torch.equal(a, b)
