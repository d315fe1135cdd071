"""Forward and data gradient of the 3 x 3 x 3 convolutions for every channel count they
take, at the edges and remainders of the output tile, with skip tensors, outputs off
an 8-byte boundary and activations that are zero, negative, infinite or NaN, against
an FP64 sum on the CPU.

Products of BF16 operands are exact in FP32, so the result is the BF16 rounding of an
FP32 sum of at most K = 27 C + 1 terms, itself within e = K 2^-24 sum |x w| of the exact
one; rounding is monotone, so it lies between the roundings of the exact sum -+ e."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _bf(a):
    return torch.tensor(np.asarray(a)).to(torch.float32).to(torch.bfloat16)


def _f(t):
    return t.to(torch.float64).numpy()


def _put(t, shift=0):
    buf = torch.empty(t.numel() + shift, dtype=t.dtype, device="cuda")
    buf[shift:] = t.reshape(-1).to("cuda")
    return buf[shift:]


def _p(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def _conv(x, w, mirror):
    """sum_{tap, c} x[p + o(tap)][c] w[n][tap][c] (offsets negated if mirror), zero outside."""
    D, H, W, _ = x.shape
    xp = np.pad(x, ((1, 1), (1, 1), (1, 1), (0, 0)))
    out = np.zeros((D, H, W, w.shape[0]))
    for t in range(27):
        a, b, c = (2 - t // 9, 2 - (t // 3) % 3, 2 - t % 3) if mirror else (t // 9, (t // 3) % 3, t % 3)
        out += xp[a:a + D, b:b + H, c:c + W] @ w[:, t].T
    return out


def _check(name, got, ref, mag, k, relu=0):
    e = k * 2.0 ** -24 * mag
    lo, hi = _f(_bf(ref - e)), _f(_bf(ref + e))
    if relu:
        lo, hi = np.maximum(lo, 0.0), np.maximum(hi, 0.0)
    print("%s: %d of %d outside" % (name, int(((got < lo) | (got > hi)).sum()), got.size), flush=True)
    assert ((got >= lo) & (got <= hi)).all()



DIMS = [(1, 1, 1), (2, 8, 16), (3, 9, 17), (5, 7, 33)]


@pytest.mark.parametrize("c1,c2,cout,dims,shift", [
    (c1, c2, n, DIMS[(i + j) % 4], (i + j) % 3)
    for i, (c1, c2) in enumerate([(16, 0), (8, 8), (32, 0), (32, 16), (64, 0), (56, 24), (64, 32)])
    for j, n in enumerate([16, 32, 64])])
def test_forward(c1, c2, cout, dims, shift):
    from paper_2512_18863_amd.learned import Vol, _lib
    print("conv3d fwd", c1, c2, cout, dims, shift, flush=True)
    lib, rng, c = _lib(), np.random.default_rng(c1 + 3 * cout), c1 + c2
    x = _bf(rng.normal(size=dims + (c,)))
    w, bias = rng.normal(size=(cout, 27, c)).astype(np.float32), rng.normal(size=cout).astype(np.float32)
    s = torch.cuda.current_stream().cuda_stream
    wg, bg = torch.tensor(w, device="cuda"), torch.tensor(bias, device="cuda")
    wt = torch.zeros(cout * lib.pdrt_conv3d_kpad(c), dtype=torch.bfloat16, device="cuda")
    wd = torch.zeros(c * lib.pdrt_conv3d_kpad(cout), dtype=torch.bfloat16, device="cuda")
    assert lib.pdrt_conv3d_prepare_weights(cout, c, _p(wg), _p(wt), _p(wd), s) == 0
    x1, x2 = _put(x[..., :c1].contiguous()), _put(x[..., c1:].contiguous()) if c2 else None
    vol, y = Vol(*dims), _put(torch.full(dims + (cout,), 9.0, dtype=torch.bfloat16), shift)
    wr = _f(_bf(w))
    ref, mag = _conv(_f(x), wr, False) + bias, _conv(np.abs(_f(x)), np.abs(wr), False) + np.abs(bias)
    for relu in (0, 1):
        assert lib.pdrt_conv3d_forward(ctypes.byref(vol), c1, c2, _p(x1), _p(x2), cout, _p(wt), _p(bg), relu, _p(y),
                                       s) == 0
        got = _f(y.cpu()).reshape(ref.shape)
        _check("relu %d" % relu, got, ref, mag, 27 * c + 1, relu)


@pytest.mark.parametrize("cout,c1,c2,dims,shift", [
    (cout, c1, c2, DIMS[(i + j) % 4], (i + j) % 3)
    for i, cout in enumerate([16, 32, 48, 64])
    for j, (c1, c2) in enumerate([(16, 0), (24, 8), (32, 16), (64, 0), (64, 32)])])
def test_data_gradient(cout, c1, c2, dims, shift):
    from paper_2512_18863_amd.learned import Vol, _lib
    print("conv3d dgrad", cout, c1, c2, dims, shift, flush=True)
    lib, rng, c = _lib(), np.random.default_rng(c1 + 5 * cout), c1 + c2
    dy, act = _bf(rng.normal(size=dims + (cout,))), _bf(rng.normal(size=dims + (cout,)))
    flat = act.reshape(-1)
    flat[:6] = torch.tensor([0.0, -0.0, float("inf"), float("nan"), -float("nan"), 1e-40], dtype=torch.bfloat16)
    w = rng.normal(size=(cout, 27, c)).astype(np.float32)
    s = torch.cuda.current_stream().cuda_stream
    wg = torch.tensor(w, device="cuda")
    wt = torch.zeros(cout * lib.pdrt_conv3d_kpad(c), dtype=torch.bfloat16, device="cuda")
    wd = torch.zeros(c * lib.pdrt_conv3d_kpad(cout), dtype=torch.bfloat16, device="cuda")
    assert lib.pdrt_conv3d_prepare_weights(cout, c, _p(wg), _p(wt), _p(wd), s) == 0
    dyg, ag, vol = _put(dy), _put(act), Vol(*dims)
    wr = np.ascontiguousarray(_f(_bf(w)).transpose(2, 1, 0))  # [ci][tap][co]
    for masked in (False, True):
        g = np.where(_f(act) > 0, _f(dy), 0.0) if masked else _f(dy)
        ref, mag = _conv(g, wr, True), _conv(np.abs(g), np.abs(wr), True)
        d1 = _put(torch.full(dims + (c1,), 9.0, dtype=torch.bfloat16), shift)
        d2 = _put(torch.full(dims + (c2,), 9.0, dtype=torch.bfloat16), shift) if c2 else None
        assert lib.pdrt_conv3d_backward_data(ctypes.byref(vol), cout, _p(dyg), _p(ag) if masked else None, c1, c2,
                                             _p(wd), _p(d1), _p(d2), s) == 0
        got = [_f(d1.cpu()).reshape(dims + (c1,))] + ([_f(d2.cpu()).reshape(dims + (c2,))] if c2 else [])
        _check("masked %d" % masked, np.concatenate(got, axis=-1), ref, mag, 27 * cout + 1)
