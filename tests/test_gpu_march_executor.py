"""Who computes the march's sums where the library has chosen the scan's order
(march_scan = None, few rays inside the field limits) but a launch marches more rays than
that: a geometry cache's whole planes, rectangles widened by fluence corrections.  The
same bits as the scan's, and not slower than the better of the two forms asked for; the
FP64 path, which marches whole planes, chooses by those."""
import numpy as np
import pytest
import torch

from paper_2512_18863_amd import engine as E
from paper_2512_18863_amd import inputs
from tests.test_gpu_parity import _say, _t

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _case(n_taps, n_cp, shape, corr=False, mode=inputs.WEPL_PER_RAY, spacing=3.0, gantry=None):
    c = inputs.tiny_case(seed=n_taps + n_cp, n_taps=n_taps, n_cp=n_cp, shape=shape, spacing=spacing, field=40.0,
                         wepl_mode=mode, gantry=gantry)
    if corr:
        c.machine = inputs.with_fluence_corrections(c.machine)
    return c


# (taps, control points, grid, corrections, depth mode, voxel size): one segment of planes,
# two, and more planes than eight segments of 32
CASES = [
    (61, 60, (8, 30, 30), False, inputs.WEPL_PER_RAY, 3.0), (31, 90, (8, 30, 31), True, inputs.WEPL_PER_RAY, 3.0),
    (41, 60, (5, 8, 8), True, inputs.WEPL_PER_RAY, 3.0), (61, 40, (3, 200, 200), False, inputs.WEPL_PER_RAY, 2.5),
    (31, 90, (8, 30, 31), True, inputs.WEPL_CENTRAL_AXIS, 3.0),
]


@pytest.mark.parametrize("n_taps,n_cp,shape,corr,mode,d", CASES,
                         ids=["%d-%d-%dx%dx%d-%d-%d" % (c[:2] + c[2] + c[3:5]) for c in CASES])
def test_same_bits_as_the_scan(n_taps, n_cp, shape, corr, mode, d):
    c = _case(n_taps, n_cp, shape, corr, mode, d)
    eng, scan = (E.DoseEngine(c, march_scan=m) for m in (None, True))
    _say("march executor n %d, %d control points, planes %d x %d x %d" % (n_taps, n_cp, eng.Nk, eng.Nu, eng.Nv))
    p, w = (_t(c.leaves), _t(c.jaws), _t(c.mu)), _t(np.random.default_rng(1).uniform(size=c.shape))
    d0, g0 = scan.forward(*p).clone(), scan.backward(*p, w)
    assert torch.equal(eng.forward(*p), d0)
    assert all(torch.equal(a, b) for a, b in zip(eng.backward(*p, w), g0))
    eng.build_cache("fp32")
    assert torch.equal(eng.forward(*p), d0)
    assert all(torch.equal(a, b) for a, b in zip(eng.backward(*p, w), g0))


def _time(names, f, reps=6):
    f()
    best = float("inf")
    for _ in range(reps):
        E.profile_begin(256)
        f()
        r = E.profile_end()
        best = min(best, sum(r[n][1] for n in names))
    return best


@pytest.mark.parametrize("what", ["cache", "corrected", "fp64"])
def test_not_slower_than_either_form(what):
    c = _case(31 if what == "corrected" else 61, 90 if what == "corrected" else 40, (64, 96, 96), what == "corrected")
    p, w = (_t(c.leaves), _t(c.jaws), _t(c.mu)), torch.ones(c.shape, device="cuda")
    ms = {}
    for form in (None, False, True):
        eng = E.DoseEngine(c, march_scan=form, with_f64=what == "fp64")
        p64 = [x.double() for x in p]
        ms[form] = {"cache": lambda: _time(["march_geometry"], lambda: eng.build_cache("fp32")),
                    "corrected": lambda: _time(["march", "march_adj"], lambda: (eng.forward(*p), eng.backward(*p, w))),
                    "fp64": lambda: _time(["march"], lambda: eng.forward_f64(*p64), 3)}[what]()
    _say("march %s: chosen %.4f ms, serial %.4f, scan %.4f" % (what, ms[None], ms[False], ms[True]))
    assert ms[None] <= 1.35 * min(ms[False], ms[True])
