"""The node arithmetic's square root, reciprocal and corrected-rate quotient on
the GPU (tests/c/node_probe, built by __graft_entry__.build()), against exact
residuals: products are taken in two doubles (Dekker), so an error is known far
below a unit in the last place.

Bounds, in units in the last place.  The hardware estimates of 1/x and 1/sqrt(x)
are good to e = 2^-23 relative (2^29 units of a double, as documented).
  reciprocal: one third-order step leaves e^3 = 2^-69 relative, at most 2^-16 units,
    before the last rounding: 1/2 + 2^-15;
  square root: the Goldschmidt step leaves 1.5 e^2 < 2^-45, the correction by the exact
    residual its square, below 2^-89: 1/2 + 2^-30;
  quotient: the estimate is within 3 units, and the correction by its residual leaves
    2^-52 of that: 1/2 + 2^-30.
"""
import os
import subprocess

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BIN = os.path.join(ROOT, "tests", "c", "node_probe")
N = 1 << 21


def two_product(a, b):
    """a b = p + q exactly (no overflow or underflow in the splits)."""
    def split(v):
        c = 134217729.0 * v
        hi = c - (c - v)
        return hi, v - hi
    p = a * b
    ah, al = split(a)
    bh, bl = split(b)
    return p, ((ah * bh - p) + ah * bl + al * bh) + al * bl


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    if not os.path.exists(BIN):
        pytest.fail("tests/c/node_probe is not built; run __graft_entry__.build()")
    d = tmp_path_factory.mktemp("node")
    rng = np.random.default_rng(2303)
    tiny = np.arange(N // 16) * 2.0 ** -52
    x = 1.0 + 3.0 * rng.random(N)
    x[:N // 16] = 1.0 + tiny                    # just above 1, just below 4, around 2
    x[N // 16:N // 8] = 4.0 - 2.0 ** -51 - 4 * tiny
    x[N // 8:3 * N // 16] = 2.0 - tiny
    den = np.exp2(rng.uniform(-20, 20, N))
    den[:N // 2] = rng.uniform(0.5, 2.0, N // 2)
    den[:N // 16] = 1.0 + tiny
    den[N // 16:N // 8] = 2.0 - tiny
    den[N // 8:N // 8 + 400] = np.exp2(np.arange(-200, 200))
    u = rng.uniform(0.0, 0.99999, N)
    u[:N // 4] = np.exp2(rng.uniform(-40, -1, N // 4))
    u[:8] = 0.0
    t = np.exp2(rng.uniform(-40, 20, N))
    t[-64:] = np.exp2(np.linspace(21, 500, 64))
    np.concatenate([np.int64([N]).view(np.float64), x, den, u, t]).tofile(d / "in")
    r = subprocess.run([BIN, str(d / "in"), str(d / "out")], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr
    out = np.fromfile(d / "out").reshape(5, N)
    return dict(x=x, den=den, u=u, t=t, root=out[0], recip=out[1], top=out[2], bottom=out[3], rate=out[4])


def _worst(err, what, bound):
    w = float(np.max(np.abs(err)))
    print(f"[node math] {what}: worst {w:.9f} units in the last place, {np.mean(np.abs(err) > 0.5):.2e} above 1/2",
          flush=True)
    assert w < bound, w


def test_square_root(probe):
    g, x = probe["root"], probe["x"]
    p, q = two_product(g, g)
    _worst(((x - p) - q) / (2.0 * g) / np.spacing(g), "square root", 0.5 + 2.0 ** -30)


def test_reciprocal(probe):
    r, d = probe["recip"], probe["den"]
    p, q = two_product(r, d)
    _worst(((1.0 - p) - q) / d / np.spacing(r), "reciprocal", 0.5 + 2.0 ** -15)


def test_corrected_rate(probe):
    w, num, den = probe["rate"], probe["top"], probe["bottom"]
    assert np.all(den > 0) and np.all(num > 0)
    p, q = two_product(w, den)
    _worst(((num - p) - q) / den / np.spacing(w), "corrected rate", 0.5 + 2.0 ** -30)
