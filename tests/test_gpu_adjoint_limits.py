"""The adjoint convolution of openings exactly at the field limits, whose rectangles are one
pixel wider than a multiple of 16: one row and column of tiles more than openings a little
inside, for which the piece size is chosen too.  A rectangle of 33 pixels fits the piece of
47 and costs no more (in pieces of two tiles it took twice the time)."""
import pytest
import torch

from tests.test_gpu_conv_planes import _case
from tests.test_gpu_parity import _say
from tests.test_gpu_small_openings import _time

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("conv", ["fp32", "bf16"])
@pytest.mark.parametrize("n_taps", [15, 31])
def test_openings_at_the_limits(n_taps, conv):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_18863_amd import inputs
    from paper_2512_18863_amd.engine import DoseEngine
    t = []
    for half in (16, 23):
        c = _case(n_taps, half, half, half, n_cp=60)
        c.jaws, c.depth_step = inputs.jaws_square(60, 2.5 * half, 2.5 * half), 4.0
        eng = DoseEngine(c, conv=conv)
        # (per plane: the grid follows the field)
        t.append(_time(eng, c, ["conv_mfma_%s_adj" % ("f32" if conv == "fp32" else "bf16")]) / eng.Nk)
    _say("%s adjoint, n %d, a plane of 60 control points: 33 x 33 %.5f ms, 47 x 47 %.5f" % ((conv, n_taps) + tuple(t)))
    assert t[0] <= 1.2 * t[1]
