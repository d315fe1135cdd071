"""The ray march's form as asked for: march_scan = False (PDRT_MARCH_SERIAL, the value of a
zeroed spec) is one thread per ray whatever the number of rays, so that a control point's
dose does not depend on how many others share its beam; True the scan; None the library's
choice, which for few rays is the scan."""
import ctypes

import pytest
import torch

from paper_2512_18863_amd import engine as E
from paper_2512_18863_amd import inputs
from tests.test_abi import _structs


@pytest.mark.gpu
@pytest.mark.parametrize("n_taps", [13, 31])
def test_serial_form_can_be_asked_for(n_taps):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests.test_gpu_parity import _say, _t, subset
    # as many control points as march serially by themselves, and three of them alone
    c = inputs.tiny_case(seed=91, n_taps=n_taps, shape=(8, 24, 24), spacing=5.0, field=100.0, n_cp=60)
    few = subset(c, [4, 17, 40])
    _say("march form, n %d" % n_taps)
    p = _t(few.leaves), _t(few.jaws), _t(few.mu)
    default, serial, scan = (E.DoseEngine(few, march_scan=m).forward(*p) for m in (None, False, True))
    assert torch.equal(default, scan) and not torch.equal(serial, scan)
    mu = torch.zeros(60, device="cuda")
    mu[[4, 17, 40]] = p[2]
    all_cps = _t(c.leaves), _t(c.jaws), mu
    assert torch.equal(E.DoseEngine(c).forward(*all_cps), serial)
    eng = E.DoseEngine(few, march_scan=False)
    eng.build_cache("fp32")
    assert torch.equal(eng.forward(*p), serial)


def test_march_values_of_the_abi():
    g, b, s, _keep = _structs(inputs.config_c0())
    assert s.march_scan == E.MARCH_SERIAL  # a zeroed spec
    for value, valid in ((-1, False), (E.MARCH_SERIAL, True), (E.MARCH_SCAN, True), (E.MARCH_AUTO, True), (3, False)):
        s.march_scan = value
        assert (E.lib().pdrt_workspace_bytes(ctypes.byref(g), ctypes.byref(b), ctypes.byref(s), 1, 4) > 0) == valid
