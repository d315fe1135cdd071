"""Corrected plans whose openings are far smaller than the field limits, by which the host
counts the rays of a march and sizes its grid: the workgroups without rays cost next to
nothing (the march of the same rays under narrower limits is the measure), and the form
chosen is not slower than the better of the two asked for."""
import pytest
import torch

from paper_2512_18863_amd import inputs
from tests.test_gpu_parity import _say
from tests.test_gpu_small_openings import _time

pytestmark = pytest.mark.gpu


def _case(field, n_cp=60):
    c = inputs.tiny_case(seed=2, n_taps=21, n_cp=n_cp, shape=(48, 64, 72), spacing=5.0, field=field)
    c.machine = inputs.with_fluence_corrections(c.machine)
    c.jaws = inputs.jaws_square(n_cp, 12.0, 12.0)
    return c


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


NAMES = ["march", "march_adj"]


def test_form_chosen():
    from paper_2512_18863_amd.engine import DoseEngine
    c = _case(60.0)
    t = [_time(DoseEngine(c, march_scan=m), c, NAMES) for m in (None, False, True)]
    _say("corrected march of 24 x 24 mm openings: chosen %.4f ms, serial %.4f, scan %.4f" % tuple(t))
    assert t[0] <= 1.25 * min(t)


def test_wide_limits_cost_nothing():
    from paper_2512_18863_amd.engine import DoseEngine
    t = []
    for field in (60.0, 32.0):
        c = _case(field)
        t.append(_time(DoseEngine(c, march_scan=True), c, NAMES))
    _say("corrected march of 24 x 24 mm openings as a scan: limits 120 mm %.4f ms, 64 mm %.4f" % tuple(t))
    assert t[0] <= 1.25 * t[1]
