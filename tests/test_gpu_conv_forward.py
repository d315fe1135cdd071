"""The register-resident forward convolution at the edges of its forms: rectangles of one
to four row blocks, one column group and several, several chunks, odd offsets, every
kernel width class, few and many items.  Dose against the FP64 oracle: FP32 <= 1e-5 of
max, BF16 <= 2^-8 of max (the bars of the other forward tests).

The reads of tap runs are modelled on the CPU: every run a lane can ask for, after its
move to the margins, lies in its row and holds the taps it stands for."""
import copy

import numpy as np
import pytest
import torch

from paper_2512_18863_amd import inputs

# conv_fwd_reg.hip: half-width limit, tap origin and words of a row
MAX_H, GROUP = 31, 32
OFF = MAX_H + 9
WORDS = (OFF + MAX_H + 10 + 1) // 2


@pytest.mark.parametrize("h", range(1, MAX_H + 1))
def test_tap_runs_model(h):
    taps = np.arange(1.0, h + 2.0)                       # K[|d|], distinct and non-zero
    copies = np.zeros((2, 2 * WORDS))
    for d in range(-h, h + 1):                           # copy 1 holds element x at x - 1
        copies[0, OFF + d] = copies[1, OFF + d - 1] = taps[abs(d)]
    for d0 in range(-(h + 3 * GROUP + 46), h + 3 * GROUP + 47):   # c - j of a run's first tap
        x, x0, x1 = d0 + OFF, OFF - h - 9, OFF + h + 1
        if x < x0 + 1:
            x = x0 + ((x ^ x0) & 1)
        if x > x1:
            x = x1 + ((x ^ x1) & 1)
        word = x >> 1
        assert 0 <= word and word + 3 < WORDS
        run = copies[x & 1, 2 * word:2 * word + 8]
        want = [taps[abs(d)] if abs(d) <= h else 0.0 for d in range(d0, d0 + 8)]
        assert np.array_equal(run, want)


# (kernel width, jaw half-widths in pixels along u and v, field limit in pixels, control points)
CASES = [
    (13, 0.4, 3.3, 6, 3), (13, 7.4, 7.6, 8, 3), (15, 8.3, 15.4, 16, 5), (31, 15.7, 16.4, 17, 3), (33, 20.2, 24.4, 25, 3),
    (61, 24.6, 31.8, 32, 2), (63, 13.3, 13.3, 14, 3), (21, 32.6, 40.3, 41, 2), (13, 52.2, 10.4, 53, 2),
    (15, 20.0, 20.0, 5, 2), (13, 3.3, 5.2, 6, 90),
]


@pytest.mark.gpu
@pytest.mark.parametrize("n_taps,ju,jv,limit,n_cp", CASES, ids=["%d-%g-%g-%d-%d" % c for c in CASES])
def test_forward_forms(n_taps, ju, jv, limit, n_cp):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_18863_amd.engine import DoseEngine
    from tests.test_gpu_parity import TOL_FWD, _rel_err, _say, _t, oracle_dose
    d = 2.5
    c = inputs.tiny_case(seed=n_taps, n_cp=n_cp, n_taps=n_taps, shape=(30, 9, 8), spacing=d, field=limit * d,
                         n_leaf=14, leaf_width=2.0 * max(jv, 4.0) * d / 14)
    c = copy.copy(c)
    rng = np.random.default_rng(n_taps)
    c.jaws = inputs.jaws_square(n_cp, ju * d, jv * d) + rng.uniform(-0.3, 0.3, size=(n_cp, 1)) * d  # shifted openings
    c.leaves = inputs.random_apertures(n_cp, 14, max(ju * d, 1.0), seed=3, max_gap=2.0 * ju * d)
    ref, m, _ = oracle_dose(c)
    for conv, tol in (("fp32", TOL_FWD), ("bf16", 2.0 ** -8)):
        eng = DoseEngine(c, conv=conv)
        lv, jw, mu = _t(c.leaves), _t(c.jaws), _t(c.mu)
        a, b = eng.forward(lv, jw, mu), eng.forward(lv, jw, mu)
        e = _rel_err(a.cpu().numpy().astype(np.float64), ref)
        _say("forward %s n %d, box %g x %g, planes %d x %d: %.2e" % (conv, n_taps, ju, jv, eng.Nu, eng.Nv, e))
        assert torch.equal(a, b)
        assert e <= tol
