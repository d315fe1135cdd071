"""The forward back-projection on thin grids under wide planes, where a voxel column's z
reach a window of the beam-frame row only: windows of one to four 64-wide pieces cut by
either end of the plane, z steps unlike the pixel, several z chunks per column, planes of
193 to 256 pixels with and without a window.  Dose against the FP64 oracle, 1e-5 of max in
FP32 and 1e-12 in FP64 (the bars of the other forward tests); and the time does not follow
the width of the plane."""
import copy

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


# (nz, step along z, lateral field, kernel width, shift of the grid along z)
CASES = [
    (1, 2.5, 100.0, 3, 0.0), (16, 2.5, 190.0, 15, 5.0), (40, 1.0, 240.0, 3, -180.0), (64, 2.5, 250.0, 3, 200.0),
    (100, 2.5, 330.0, 3, -3.0), (200, 2.5, 250.0, 3, 0.0), (200, 1.2, 330.0, 3, 90.0), (30, 6.0, 230.0, 3, 1.0),
    (128, 2.5, 250.0, 3, 240.0), (250, 2.5, 330.0, 5, 0.0),
]


@pytest.mark.parametrize("nz,sz,field,n_taps,shift", CASES, ids=["%d-%g-%g-%d-%g" % c for c in CASES])
def test_window_forms(nz, sz, field, n_taps, shift):
    from paper_2512_18863_amd.engine import DoseEngine
    c = inputs.tiny_case(seed=nz + 3, n_cp=3, n_taps=n_taps, shape=(nz, 8, 9), spacing=2.5, field=field, n_leaf=12,
                         leaf_width=2.0 * field / 12)
    c = copy.copy(c)
    c.spacing = (2.5, 2.5, sz)
    c.origin = (c.origin[0], c.origin[1], -0.5 * (nz - 1) * sz + shift)
    c.lat_step = c.depth_step = 2.5
    # apertures as wide as the field, so that every part of the row carries dose
    c.jaws = inputs.jaws_square(3, field, field)
    c.leaves = np.stack([np.full((3, 12), -field), np.full((3, 12), field)], axis=1)
    eng = DoseEngine(c, with_f64=True)
    lv, jw, mu = _t(c.leaves), _t(c.jaws), _t(c.mu)
    ref, _, rho = oracle_dose(c)
    got = eng.forward(lv, jw, mu)
    eng.set_density_f64(_t(rho, torch.float64))
    f64 = eng.forward_f64(lv.double(), jw.double(), _t(c.mu, torch.float64))
    e, e64 = _rel_err(got.cpu().numpy().astype(np.float64), ref), _rel_err(f64.cpu().numpy(), ref)
    _say("gather window nz %d sz %g, planes %d x %d x %d: %.2e, FP64 %.2e" % (nz, sz, eng.Nk, eng.Nu, eng.Nv, e, e64))
    assert (ref > 0.01 * ref.max()).mean() > 0.5
    assert e <= TOL_FWD and e64 <= 1e-12
    assert torch.equal(DoseEngine(c, max_cp_batch=2).forward(lv, jw, mu), got)


def test_time_follows_the_window_not_the_plane():
    from paper_2512_18863_amd import engine as E
    ms = {}
    for field in (50.0, 230.0):  # along z only: every control point reaches the same columns
        c = inputs.tiny_case(seed=5, n_cp=60, n_taps=7, shape=(16, 96, 96), spacing=2.5, field=50.0, n_leaf=12,
                             leaf_width=2.0 * field / 12)
        c = copy.copy(c)
        c.field_limit = (50.0, field)
        eng = E.DoseEngine(c)
        p = _t(c.leaves), _t(c.jaws), _t(c.mu)
        best = float("inf")
        for _ in range(8):
            E.profile_begin(64)
            eng.forward(*p)
            best = min(best, E.profile_end()["gather"][1])
        _say("gather under %d x %d planes: %.4f ms" % (eng.Nu, eng.Nv, best))
        ms[eng.Nv] = best
    narrow, wide = (ms[k] for k in sorted(ms))
    assert wide <= 1.6 * narrow
