"""Openings far smaller than the field limits, by which the host sizes the launches: the
adjoint convolution's pieces of three by three and four by four tiles hold rectangles of
one, two and three tiles (every pixel against FP64, the bars of the planes' test) and
cost less than full ones."""
import pytest
import torch

from tests.test_gpu_conv_planes import _case, _error
from tests.test_gpu_parity import _say, _t

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# limits of three and of four tiles across; openings of 1, 2, 3 tiles a side, or of both
@pytest.mark.parametrize("n_taps,limit", [(13, 23), (61, 23), (21, 31), (61, 31)])
@pytest.mark.parametrize("ju,jv", [(4.2, 4.4), (6.6, 12.2), (14.2, 13.3), (5.1, 20.2), (20.3, 20.4)])
def test_adjoint_planes(n_taps, limit, ju, jv):
    c = _case(n_taps, ju, jv, limit)
    for conv, tol in (("fp32", 5e-6), ("bf16", 2.0 ** -8)):
        e, planes, box = _error(c, conv, "adjoint")
        _say("%s n %d, planes %d x %d x %d, boxes up to %d x %d: %.2e" % ((conv, n_taps) + planes +
                                                                         (box[0], box[1], e)))
        assert e <= tol


def _time(eng, c, names, reps=8):
    from paper_2512_18863_amd import engine as E
    p, w = (_t(c.leaves), _t(c.jaws), _t(c.mu)), torch.ones(c.shape, device="cuda")
    best = float("inf")
    for _ in range(reps):
        E.profile_begin(256)
        eng.forward(*p)
        eng.backward(*p, w)
        r = E.profile_end()
        best = min(best, sum(r[n][1] for n in names))
    return best


def test_adjoint_cost_of_small_openings():
    """One tile of nine is multiplied, not all of them."""
    from paper_2512_18863_amd.engine import DoseEngine
    small, full = (_case(61, j, j, 23, n_cp=60) for j in (5.0, 22.0))
    t = [_time(DoseEngine(c), c, ["conv_mfma_f32_adj"]) for c in (small, full)]
    _say("adjoint of 60 control points, limits 23 px: openings of 10 px %.4f ms, of 44 px %.4f ms" % tuple(t))
    assert t[0] <= 0.8 * t[1]
