"""Table builds away from the default grid, against the oracle's inversion: the
smallest grids, ranges far into both tails, and pair tables whose Bessel
functions lie inside and past the interpolated range."""
import numpy as np
import pytest
from scipy.integrate import quad
from scipy.special import kve

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu


def emission_tail(chi, q):
    """The part of the emission spectrum above logit(delta) - ln chi = q, minus its slope in q, and the whole
    spectrum, by adaptive quadrature in w = ln(y) / 3 (the reference where 1 - r < 5e-5: the oracle's inversion ends at 1e-7 of
    the tail there)."""
    def f(w):
        y = np.exp(3 * w)
        omd = 1 / (1 + 1.5 * chi * y)
        ki13 = quad(lambda t: np.exp(-y * (np.cosh(t) - 1)) * np.cosh(t / 3) / np.cosh(t), 0,
                    np.arccosh(1 + 60 / y), epsabs=0, epsrel=1e-12, limit=400)[0]
        return ((omd + 1 / omd) * kve(2 / 3, y) - ki13) * np.exp(-y) * y * omd * omd

    def over(a, b, n):
        e = np.linspace(a, b, n + 1)
        return sum(quad(f, lo, hi, epsabs=0, epsrel=1e-11)[0] for lo, hi in zip(e[:-1], e[1:]))
    w = (q - np.log(1.5)) / 3
    return over(w, w + 1.0, 20), f(w) / 3, f(-14.0) + over(-14.0, 1.6, 32)


@pytest.mark.parametrize("cfg", [
    dict(rad_rows=4, rad_cols=4, pair_rows=4, pair_cols=4, f64_refine=1),
    dict(rad_rows=5, rad_cols=513, pair_rows=6, pair_cols=515, f64_refine=3, rate_nodes=64),
    dict(rad_chi_min=1e-6, rad_chi_max=1e6, rad_x_min=-20.0, rad_x_max=30.0, pair_chi_min=1e-3, pair_chi_max=1e6,
         pair_x_min=-30.0, rad_rows=24, pair_rows=24, f64_refine=2),
])
def test_nodes_vs_oracle(cfg, orc):
    _, sf = need_gpu()
    tabs = sf.Tables(sf.default_table_cfg(**cfg))
    g = tabs.geometry()
    rng = np.random.default_rng(4)
    for p, name in ((0, "rad"), (1, "pair")):
        for bits in (32, 64):
            T = tabs.export(f"cdf{bits}_{name}").astype(np.float64)
            rows, cols = T.shape
            hs = (g[f"s1_{p}"] - g[f"s0_{p}"]) / (rows - 1)
            hx = (g[f"x1_{p}"] - g[f"x0_{p}"]) / (cols - 1)
            for n in range(24):  # corners first
                i = (0, rows - 1)[n & 1] if n < 4 else int(rng.integers(0, rows))
                j = (0, cols - 1)[n >> 1] if n < 4 else int(rng.integers(0, cols))
                chi, x = np.exp(g[f"s0_{p}"] + i * hs), g[f"x0_{p}"] + j * hx
                r, rc = 1 / (1 + np.exp(-x)), 1 / (1 + np.exp(x))
                if p == 0 and x > 10.0:
                    tail, slope, total = emission_tail(chi, T[i, j])
                    q = T[i, j] + (tail - rc * total) / slope
                elif p == 0:
                    d, omd = orc.sample_rad_r2(chi, r, rc)
                    q = np.log(d) - np.log(omd) - np.log(chi)
                else:
                    xi = orc.sample_pair_r(chi, r, rc=rc)
                    if not 0.0 < xi < 1.0:  # the oracle's inversion has underflowed
                        continue
                    q = np.log(xi) - np.log1p(-xi)
                # FP64: the bound the default grid's nodes are held to; FP32: half an ulp of q more
                tol = 1e-10 * max(1.0, abs(q)) + (2.0 ** -24 * abs(q) if bits == 32 else 0.0)
                assert abs(T[i, j] - q) <= tol, (bits, name, i, j, T[i, j], q)


def test_pair_rows_past_the_interpolated_range():
    """Far below threshold the pair spectrum is a Gaussian in logit xi whose
    width goes as sqrt(chi), with corrections of relative order chi.  The
    rows at chi = 1e-8 take their Bessel functions from the sums, those at 1e-7
    from the interpolation, so their ratio checks both: sqrt(10) to 1e-6 (the
    corrections, and the rounding of y - y0 ~ 1 at y ~ 3e8, a few 1e-8)."""
    _, sf = need_gpu()
    tabs = sf.Tables(sf.default_table_cfg(pair_chi_min=1e-8, pair_chi_max=1e-5, pair_rows=4, pair_cols=93,
                                          f64_refine=1, rad_rows=4, rad_cols=4))
    T = tabs.export("cdf64_pair")
    assert np.allclose(T[1, :-1] / T[0, :-1], np.sqrt(10.0), rtol=1e-6)
    assert np.allclose(T[2, :-1] / T[1, :-1], np.sqrt(10.0), rtol=1e-5)
