"""Weight and bias gradients of the 3 x 3 x 3 convolutions (the matrix-core kernel and
its rule) against an FP64 sum on the CPU, at tile edges and remainders of every
dimension, partial channel tiles, one and more splits than tiles, and the scalar
kernel for buffers that are not 16-byte aligned.

Products of BF16 operands are exact in FP32, so the only error is that of FP32 sums of
N = D H W terms in some order: at most N 2^-24 sum |g x| to first order."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _reference(x, g):
    """(dw [co][27][ci], db [co]) in FP64 for x [D][H][W][ci], g [D][H][W][co]."""
    D, H, W, _ = x.shape
    xp = np.pad(x, ((1, 1), (1, 1), (1, 1), (0, 0)))
    dw = np.stack([np.tensordot(g, xp[t // 9:t // 9 + D, (t // 3) % 3:(t // 3) % 3 + H, t % 3:t % 3 + W],
                                axes=([0, 1, 2], [0, 1, 2])) for t in range(27)], axis=1)
    return dw, g.sum(axis=(0, 1, 2))


@pytest.mark.parametrize("dims,c1,c2,cout,act,nsplit,shift", [
    ((1, 1, 1), 16, 0, 16, True, 2, 0),
    ((3, 4, 32), 16, 0, 16, True, 2, 0),
    ((2, 5, 33), 16, 0, 32, False, 3, 0),
    ((3, 3, 31), 8, 0, 8, True, 2, 0),
    ((2, 9, 65), 32, 16, 16, True, 700, 0),
    ((2, 7, 30), 24, 16, 24, True, 4, 0),
    ((4, 8, 34), 64, 32, 32, True, 5, 0),
    ((3, 6, 20), 64, 0, 64, True, 1, 0),
    ((2, 4, 40), 32, 0, 40, False, 7, 0),
    ((2, 5, 9), 16, 0, 16, True, 3, 1),
    ((2, 5, 9), 16, 0, 12, True, 3, 0),
])
def test_weight_gradient(dims, c1, c2, cout, act, nsplit, shift):
    from paper_2512_18863_amd.learned import Vol, _lib
    print("wgrad", dims, c1, c2, cout, act, nsplit, shift, flush=True)
    lib = _lib()
    rng = np.random.default_rng(sum(dims) + c1 + cout)
    cin, n = c1 + c2, int(np.prod(dims))
    bf = lambda a: torch.tensor(a, dtype=torch.float32).to(torch.bfloat16)
    x, dy, y = (bf(rng.normal(size=dims + (c,))) for c in (cin, cout, cout))

    def put(t):  # on the GPU, `shift` elements past a 16-byte boundary
        buf = torch.empty(t.numel() + shift, dtype=t.dtype, device="cuda")
        buf[shift:] = t.reshape(-1).to("cuda")
        return buf[shift:]

    x1, dyg, yg = put(x[..., :c1].contiguous()), put(dy), put(y)
    x2 = put(x[..., c1:].contiguous()) if c2 else None
    wsb = lib.pdrt_conv3d_wgrad_ws_bytes(cout, cin, nsplit)
    guard = 64
    ws = torch.full((wsb // 4 + guard,), 7.0, dtype=torch.float32, device="cuda")
    dw = torch.empty((cout, 27, cin), dtype=torch.float32, device="cuda")
    db = torch.empty(cout, dtype=torch.float32, device="cuda")
    out = []
    for _ in range(2):
        assert lib.pdrt_conv3d_backward_weight(
            ctypes.byref(Vol(*dims)), c1, c2, x1.data_ptr(), x2.data_ptr() if c2 else None, cout, dyg.data_ptr(),
            yg.data_ptr() if act else None, nsplit, ws.data_ptr(), wsb, dw.data_ptr(), db.data_ptr(),
            torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        out.append((dw.cpu().clone(), db.cpu().clone()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])  # deterministic
    assert bool((ws[wsb // 4:] == 7.0).all())                                       # inside the workspace
    g64, x64 = dy.double().numpy(), x.double().numpy()
    if act:
        g64 = g64 * (y.float().numpy() > 0)
    rw, rb = _reference(x64, g64)
    aw, ab = _reference(np.abs(x64), np.abs(g64))
    assert np.all(np.abs(out[0][0].double().numpy() - rw) <= n * 2.0 ** -24 * aw + 1e-30)
    assert np.all(np.abs(out[0][1].double().numpy() - rb) <= n * 2.0 ** -24 * ab + 1e-30)
