"""The network's output head and its backward, eight channels at a time and one by one
(channel counts that are no multiple of 8, buffers off a 16-byte boundary), at the
block's edges in positions, with and without weight gradients, against FP64 on the CPU.

Bounds: an FP32 sum of k terms is within k 2^-24 of the sum of its terms' magnitudes;
BF16 results lie between the roundings of the exact value -+ that bound."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _p(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _bf(a):
    return torch.tensor(np.asarray(a)).to(torch.float32).to(torch.bfloat16)


@pytest.mark.parametrize("n,c,shift", [(1, 16, 0), (255, 8, 0), (256, 16, 0), (257, 24, 0), (1000, 16, 1), (700, 16, 8),
                                       (513, 1, 0), (300, 12, 0), (260, 5, 3)])
def test_head(n, c, shift):
    from paper_2512_18863_amd.learned import _lib
    print("head", n, c, shift, flush=True)
    lib, rng, s = _lib(), np.random.default_rng(n + c), torch.cuda.current_stream().cuda_stream
    f32 = lambda a: torch.tensor(np.asarray(a), dtype=torch.float32, device="cuda")
    x = _bf(rng.normal(size=(n, c)))
    xg = torch.empty(n * c + shift, dtype=torch.bfloat16, device="cuda")[shift:]
    xg.copy_(x.reshape(-1))
    hw, hb, dose, scale = f32(rng.normal(size=(2, c))), f32(rng.normal(size=2)), f32(rng.random(n)), f32([0.37])
    gp, gr = f32(rng.normal(size=n)), f32(rng.normal(size=n))
    pred, resid = torch.empty(n, device="cuda"), torch.empty(n, device="cuda")
    assert lib.pdrt_net_head(n, c, _p(xg), _p(hw), _p(hb), _p(dose), _p(scale), _p(pred), _p(resid), s) == 0
    X, H, B, D, S, G0, G1 = (t.cpu().double().numpy() for t in (x, hw, hb, dose, scale, gp, gr))
    u = 2.0 ** -24
    for got, ref, mag in ((pred, D * S + B[0] + X @ H[0], D * S + abs(B[0]) + np.abs(X) @ np.abs(H[0])),
                          (resid, B[1] + X @ H[1], abs(B[1]) + np.abs(X) @ np.abs(H[1]))):
        assert (np.abs(got.cpu().double().numpy() - ref) <= (c + 3) * u * mag).all()
    for g1 in (gr, None):
        q1 = G1 if g1 is not None else np.zeros(n)
        for want in (True, False):
            dx = torch.full((n * c + shift,), 9.0, dtype=torch.bfloat16, device="cuda")[shift:]
            ws = torch.empty(lib.pdrt_net_head_ws_bytes(n, c), dtype=torch.uint8, device="cuda")
            dh = torch.full((2 * c + 2,), 9.0, device="cuda") if want else None
            assert lib.pdrt_net_head_backward(n, c, _p(xg), _p(hw), _p(gp), _p(g1), _p(dx), _p(ws), ws.numel(), _p(dh),
                                              s) == 0
            ref = np.outer(G0, H[0]) + np.outer(q1, H[1])
            e = 3 * u * (np.abs(np.outer(G0, H[0])) + np.abs(np.outer(q1, H[1])))
            got = dx.cpu().double().numpy().reshape(n, c)
            assert (got >= _bf(ref - e).double().numpy()).all() and (got <= _bf(ref + e).double().numpy()).all()
            if want:
                r = np.concatenate([G0 @ X, q1 @ X, [G0.sum(), q1.sum()]])
                m = np.concatenate([np.abs(G0) @ np.abs(X), np.abs(q1) @ np.abs(X), [np.abs(G0).sum(), np.abs(q1).sum()]])
                assert (np.abs(dh.cpu().double().numpy() - r) <= (n + 1) * u * m).all()
