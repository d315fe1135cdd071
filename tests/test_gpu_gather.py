"""The back-projection's forward (k_gather) at the edges of its forms: planes of one to
five 64-wide pieces and wider, z chunks of one, two and three values per lane and their
remainders, control points in batches (the running sum carried between them), fans that
miss voxel columns, and a non-finite MU.  Bars as for the other forward tests: dose
<= 1e-5 of max against the FP64 oracle; a sum carried over batches is the same sum."""
import numpy as np
import pytest
import torch

from paper_2512_18863_amd import inputs
from tests.test_gpu_parity import TOL_FWD, _rel_err, _say, _t, oracle_dose

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (nz, lateral field, kernel width): Nv = 2 ceil(field / 2.5 + h) + 1 with 2.5 mm pixels
CASES = [
    (1, 10.0, 3), (64, 70.0, 13), (65, 77.5, 3), (128, 140.0, 31), (129, 150.0, 15), (193, 230.0, 3),
    (40, 310.0, 15), (70, 330.0, 3),
]


@pytest.mark.parametrize("nz,field,n_taps", CASES, ids=["%d-%g-%d" % c for c in CASES])
def test_gather_forms(nz, field, n_taps):
    from paper_2512_18863_amd.engine import DoseEngine
    c = inputs.tiny_case(seed=nz, n_cp=5, n_taps=n_taps, shape=(nz, 9, 7), spacing=2.5, field=field, n_leaf=12,
                         leaf_width=2.0 * field / 12)
    eng = DoseEngine(c)
    _say("gather nz %d, planes %d x %d x %d" % (nz, eng.Nk, eng.Nu, eng.Nv))
    lv, jw, mu = _t(c.leaves), _t(c.jaws), _t(c.mu)
    got = eng.forward(lv, jw, mu)
    assert _rel_err(got.cpu().numpy().astype(np.float64), oracle_dose(c)[0]) <= TOL_FWD
    for batch in (1, 2):
        assert torch.equal(DoseEngine(c, max_cp_batch=batch).forward(lv, jw, mu), got)
    mu[1] = float("nan")
    assert bool(torch.isnan(eng.forward(lv, jw, mu)).all())


def test_gather_skips_and_batches_of_many_control_points():
    from paper_2512_18863_amd.engine import DoseEngine
    # 70 control points (two lists of at most 64), a narrow fan that misses most columns
    c = inputs.tiny_case(seed=9, n_cp=70, n_taps=5, shape=(6, 60, 60), spacing=5.0, field=15.0)
    lv, jw, mu = _t(c.leaves), _t(c.jaws), _t(c.mu)
    eng = DoseEngine(c)
    _say("gather 70 control points, planes %d x %d x %d" % (eng.Nk, eng.Nu, eng.Nv))
    got = eng.forward(lv, jw, mu)
    assert _rel_err(got.cpu().numpy().astype(np.float64), oracle_dose(c)[0]) <= TOL_FWD
    assert torch.equal(DoseEngine(c, max_cp_batch=33).forward(lv, jw, mu), got)
