"""The ray march's form by itself (march_scan = 0): few rays take the segmented
scan, kernels of at most 11 taps and problems with more rays the serial form, and a
depth-dose table too long for the scan's LDS the serial form as well.

A route is told by its bits against march_scan = 1 (the same kernel, hence equal) and
every result is held to the FP64 oracle: 1e-5 of the largest dose, 1e-12 in FP64."""
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


def _params(c):
    return _t(c.leaves), _t(c.jaws), _t(c.mu)


# (taps, grid, spacing, control points): small and long rays (more than 256 planes, several passes)
@pytest.mark.parametrize("kw", [
    dict(seed=81, n_taps=13, shape=(9, 8, 10), spacing=6.0, field=40.0, n_cp=1),
    dict(seed=82, n_taps=33, shape=(12, 60, 50), spacing=4.0, field=45.0, n_cp=5),
    dict(seed=83, n_taps=15, shape=(3, 200, 200), spacing=2.5, field=25.0, n_cp=3),
    dict(seed=84, n_taps=15, shape=(7, 30, 31), spacing=5.0, field=25.0, n_cp=3, wepl_mode=inputs.WEPL_CENTRAL_AXIS),
], ids=["one-field", "five", "long", "central-axis"])
def test_few_rays_take_the_scan(kw):
    from paper_2512_18863_amd.engine import DoseEngine
    c = inputs.tiny_case(**kw)
    _say("march rule %s" % kw)
    eng, scan = DoseEngine(c), DoseEngine(c, march_scan=True)
    p, w = _params(c), _t(np.random.default_rng(kw["seed"]).uniform(size=c.shape))
    d = eng.forward(*p).clone()
    g = [x.clone() for x in eng.backward(*p, w)]
    assert _rel_err(d.cpu().numpy().astype(np.float64), oracle_dose(c)[0]) <= TOL_FWD
    assert torch.equal(d, scan.forward(*p))
    for a, b in zip(g, scan.backward(*p, w)):
        assert torch.equal(a, b)
    eng.build_cache("fp32")  # cached and uncached march alike
    assert torch.equal(d, eng.forward(*p))
    for a, b in zip(g, eng.backward(*p, w)):
        assert torch.equal(a, b)


# small kernels, and a plan of many control points: the two forms' sums differ in their last bits
@pytest.mark.parametrize("kw", [
    dict(seed=85, n_taps=11, shape=(12, 60, 50), spacing=4.0, field=45.0, n_cp=2),
    dict(seed=86, n_taps=13, shape=(8, 24, 24), spacing=5.0, field=100.0, n_cp=60),
], ids=["small-kernel", "many-rays"])
def test_others_stay_serial(kw):
    from paper_2512_18863_amd.engine import DoseEngine
    c = inputs.tiny_case(**kw)
    _say("march rule %s" % kw)
    p = _params(c)
    d = DoseEngine(c).forward(*p)
    assert _rel_err(d.cpu().numpy().astype(np.float64), oracle_dose(c)[0]) <= TOL_FWD
    assert not torch.equal(d, DoseEngine(c, march_scan=True).forward(*p))


def test_long_table_in_fp64_stays_serial():
    from paper_2512_18863_amd.engine import DoseEngine
    c = inputs.tiny_case(seed=87, n_taps=13, shape=(9, 8, 10), spacing=6.0, field=40.0)
    m = c.machine
    x = np.linspace(0.0, (len(m.dd) - 1) * m.dd_step, 8192)
    dd = np.interp(x, np.arange(len(m.dd)) * m.dd_step, np.asarray(m.dd))
    c = dataclasses.replace(c, machine=dataclasses.replace(m, dd=dd, dd_step=float(x[1])))
    eng = DoseEngine(c, with_f64=True)
    ref, _, rho = oracle_dose(c)
    d = eng.forward(*_params(c)).cpu().numpy().astype(np.float64)
    eng.set_density_f64(_t(rho, torch.float64))
    d64 = eng.forward_f64(*(_t(a, torch.float64) for a in (c.leaves, c.jaws, c.mu))).cpu().numpy()
    _say("8192-entry table: FP32 %.3e, FP64 %.3e" % (_rel_err(d, ref), _rel_err(d64, ref)))
    assert _rel_err(d, ref) <= TOL_FWD
    assert _rel_err(d64, ref) <= 1e-12
