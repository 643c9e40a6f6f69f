"""The FP32 main lobe of the sinc (sinc_lobe: a polynomial times the clamped
1 - t^2) against numpy's sinc: the constants are read from the kernel header and
evaluated in FP32 as the kernels do, over the lobe and beyond it."""
import re

import numpy as np

from test_sinc_poly_constants import HDR, _fma32


def test_fp32_sinc_lobe_matches_numpy():
    src = HDR.read_text()
    body = src[src.index("sinc_lobe<float>(float t) {"):]
    body = body[:body.index("\n}\n")]
    coefs = [float(re.search(r"float s = ([-+0-9.eE]+)f;", body).group(1))]
    coefs += [float(v) for v in re.findall(r"fmaf\(s, y, ([-+0-9.eE]+)f\)", body)]
    assert len(coefs) == 6 and coefs[-1] == 1.0
    t = np.linspace(-3.0, 3.0, 600_001).astype(np.float32)
    y = t * t
    s = np.full_like(y, np.float32(coefs[0]))
    for c in coefs[1:]:
        s = _fma32(s, y, np.full_like(y, np.float32(c)))
    got = s * np.clip(_fma32(-t, t, np.ones_like(t)), 0, 1)
    want = np.where(np.abs(t) < 1, np.sinc(t.astype(np.float64)), 0.0)
    # 9e-10 of the fit, six roundings of numbers up to 1 of which the later ones
    # are scaled by 1 - t^2: two units of 6e-8
    assert np.abs(got - want).max() < 1.3e-7
    assert got[300_000] == 1.0 and np.all(got[np.abs(t) >= 1] == 0)
