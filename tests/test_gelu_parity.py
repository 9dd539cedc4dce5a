"""GELU and its derivative where the short form of the bf16 kernels can go
wrong: both signs, zeros, the tails where the CDF leaves fp32's range, values
whose square overflows, infinities and NaN.  Through pf_gelu_bwd (dH = 1) and
the forward epilogue of a one-block identity layer, against scipy's erfc in
float64.  The outputs are bf16 (8 significant bits): half a unit in the last
place is at most 2^-8 of the value.  On top, the fp32 form's own error: 3e-5
of the value (the fit past its range of 10 and the rounding of x^2 in the
exponent, at |x| = 13: 2e-5), and 1e-6 absolute where
CDF and density cancel (the derivative's zero near x = -0.75), falling off
with the density; an exponential below 2^-126 flushes to zero, which the
derivative multiplies by |x| (up to 14 before the next bf16 of it is zero too)."""
import numpy as np
import pytest
from scipy.special import erfc

import synth
from tests._gpu_util import empty, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu


def _points():
    g = np.concatenate([np.linspace(-14, 14, 4001), [0.0, -0.0, 1e-30, -1e-30, 30.0, -30.0, 1e4, -1e4,
                                                      1e20, -1e20, 3e38, -3e38, np.inf, np.nan]])
    x = np.zeros(4096)
    x[:g.size] = g
    raw = synth.bf16_bits_from_f32(x.astype(np.float32))
    return synth.f32_from_bf16_bits(raw).astype(np.float64), raw


def _cdf(x):
    return 0.5 * erfc(-x / np.sqrt(2.0))


def _close(got, ref, x):
    fin = np.isfinite(x) & np.isfinite(ref)
    err = np.abs(got[fin] - ref[fin])
    density = np.exp(-0.5 * np.minimum(x[fin] ** 2, 1400.0))
    bound = (2.0 ** -8 + 3e-5) * np.abs(ref[fin]) + 1e-6 * density + 15 * 2.0 ** -126
    i = int(np.argmax(err - bound))
    assert (err <= bound).all(), (x[fin][i], got[fin][i], ref[fin][i])


def test_gelu_derivative_points():
    torch_cuda()
    from paper_2112_00029_amd import pixelfly as pf
    x, raw = _points()
    one = synth.bf16_bits_from_f32(np.ones(x.size, np.float32))
    out = empty((x.size,), "bf16")
    print("[gelu_bwd] 4096 points", flush=True)
    pf.pf_gelu_bwd(pf.PF_BF16, x.size, to_dev(one), to_dev(raw), out)
    got = to_host(out)
    with np.errstate(all="ignore"):
        ref = _cdf(x) + x * np.exp(-0.5 * x * x) / np.sqrt(2 * np.pi)
    _close(got, ref, x)
    assert np.isnan(got[np.isnan(x)]).all()


def test_gelu_forward_points():
    """X = the points (64 per row, one row each), W = I: Y_pre = X."""
    torch_cuda()
    from paper_2112_00029_amd import pixelfly as pf
    x, raw = _points()
    x, raw = x[np.isfinite(x)], raw[np.isfinite(x)]  # 0 * inf of the identity's zeros is NaN
    n = x.size // 32 * 32
    x, raw = x[:n].reshape(-1, 32), raw[:n].reshape(-1, 32)
    L = pf.pf_layout_create(32, 32, 32, 1)
    pf.pf_layout_upload(L)
    W = synth.bf16_bits_from_f32(np.eye(32, dtype=np.float32)[None])
    T = x.shape[0]
    y, pre = empty((T, 32), "bf16"), empty((T, 32), "bf16")
    print(f"[gelu forward] T={T}", flush=True)
    pf.pf_linear_fwd(L, pf.PF_BF16, T, 0, to_dev(raw), to_dev(W), None, None, y, None, pf.PF_EPI_GELU, pre)
    assert np.array_equal(to_host(pre), x)
    with np.errstate(all="ignore"):
        ref = x * _cdf(x)
    _close(to_host(y).ravel(), ref.ravel(), x.ravel())
