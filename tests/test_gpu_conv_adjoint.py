"""The adjoint convolution for outputs inside the aperture rectangle (conv_adj.hip) at the
edges of its forms: one to four tiles per piece and several pieces, rectangles one tile
smaller than their piece and larger than the field limit, odd offsets, windows cut by the
plane, every kernel width class, widened and turned rectangles.  Gradients against the
FP64 oracle: FP32 <= 1e-4 of max |g| per group, BF16 <= 2^-8 (the bars of the other
gradient tests); repeated calls agree bit for bit."""
import copy

import numpy as np
import pytest
import torch

import oracle
from paper_2512_18863_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (kernel width, jaw half-widths in pixels along u and v, field limit in pixels, corrections, collimator)
CASES = [
    (13, 0.4, 3.3, 6, False, False), (13, 7.4, 7.6, 8, False, False), (15, 8.3, 15.4, 16, False, False),
    (31, 15.7, 16.4, 17, False, False), (33, 20.2, 24.4, 25, False, False), (61, 24.6, 31.8, 32, False, False),
    (63, 13.3, 13.3, 14, False, False), (21, 32.6, 40.3, 41, False, False), (13, 52.2, 10.4, 53, False, False),
    (15, 20.0, 20.0, 5, False, False), (13, 9.3, 6.2, 10, True, False), (15, 9.3, 12.2, 13, False, True),
    (17, 8.3, 9.2, 10, True, True),
]


@pytest.mark.parametrize("n_taps,ju,jv,limit,corr,coll", CASES, ids=["%d-%g-%g-%d-%d-%d" % c for c in CASES])
def test_adjoint_forms(n_taps, ju, jv, limit, corr, coll):
    from paper_2512_18863_amd.engine import DoseEngine
    from tests.test_gpu_parity import _say, _t
    d, n_cp = 2.5, 2
    c = inputs.tiny_case(seed=n_taps, n_cp=n_cp, n_taps=n_taps, shape=(30, 9, 8), spacing=d, field=limit * d,
                         n_leaf=14, leaf_width=2.0 * max(jv, 4.0) * d / 14)
    c = copy.copy(c)
    rng = np.random.default_rng(n_taps)
    c.jaws = inputs.jaws_square(n_cp, ju * d, jv * d) + rng.uniform(-0.3, 0.3, size=(n_cp, 1)) * d
    c.leaves = inputs.random_apertures(n_cp, 14, max(ju * d, 1.0), seed=3, max_gap=2.0 * ju * d)
    if corr:
        c.machine = inputs.with_fluence_corrections(c.machine)
    if coll:
        c.collimator = rng.uniform(-45.0, 45.0, size=n_cp)
    w = rng.uniform(size=c.shape).astype(np.float32)
    m = oracle.Model(c)
    kw = {"coll": c.collimator} if coll else {}
    ref = oracle.backward(m, oracle.density(m), c.gantry, c.leaves, c.jaws, c.mu, w.astype(np.float64), **kw)
    args = (_t(c.leaves), _t(c.jaws), _t(c.mu), _t(w))
    for conv, tol in (("fp32", 1e-4), ("bf16", 2.0 ** -8)):
        eng = DoseEngine(c, conv=conv)
        got, again = eng.backward(*args), eng.backward(*args)
        for name, a, b, r in zip(("leaves", "jaws", "mu"), got, again, ref):
            e, top = np.abs(a.cpu().numpy() - r).max(), np.abs(r).max()
            _say("adjoint %s n %d, box %g x %g, planes %d x %d, %s: %.2e of %.2e" % (conv, n_taps, ju, jv, eng.Nu,
                                                                                    eng.Nv, name, e, top))
            assert torch.equal(a, b)
            assert e <= tol * top
