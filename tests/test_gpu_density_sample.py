"""Density samples of the ray march at the faces of the CT: volumes one or two voxels
thick along an axis, so that most samples have corners outside or are outside
altogether, and rays that miss the volume, against the FP64 oracle; both forms of the
march.  Forward within 1e-5 of the largest dose (FP32) and 1e-12 (FP64)."""
import dataclasses

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


@pytest.mark.parametrize("shape", [(1, 6, 7), (6, 1, 7), (6, 7, 1), (2, 2, 2), (1, 1, 9), (9, 5, 4)])
@pytest.mark.parametrize("scan", [False, True])
def test_thin_volumes(shape, scan):
    from paper_2512_18863_amd.engine import DoseEngine
    c = inputs.tiny_case(seed=sum(shape), n_cp=4, n_taps=5, shape=shape, spacing=9.0, field=40.0)
    c = dataclasses.replace(c, iso=(11.0, -7.0, 5.0))
    _say("density samples, %s, scan %d" % (shape, scan))
    eng = DoseEngine(c, with_f64=True, march_scan=scan)
    d = eng.forward(_t(c.leaves), _t(c.jaws), _t(c.mu)).cpu().numpy().astype(np.float64)
    ref, _, rho = oracle_dose(c)
    eng.set_density_f64(_t(rho, torch.float64))
    d64 = eng.forward_f64(*(_t(a, torch.float64) for a in (c.leaves, c.jaws, c.mu))).cpu().numpy()
    assert ref.max() > 0
    assert _rel_err(d, ref) <= TOL_FWD
    assert _rel_err(d64, ref) <= 1e-12
