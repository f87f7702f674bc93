"""Response spectra with the records cut into parts: record lengths at the edges
of a part and of the samples loaded ahead, few and many wavefronts, against the
oracle's stepping (1e-10 of the peak, as for whole records) and the device's own
spectra of the series one by one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("series,samples,periods", [(1, 1, 1), (2, 15, 3), (3, 16, 5), (1, 127, 40), (2, 128, 33),
                                                    (5, 257, 7), (4, 1023, 64), (3, 2001, 5), (900, 130, 37),
                                                    (2400, 40, 110)])
def test_parts_match_oracle(gpu_ctx, oracle_lib, series, samples, periods):
    rng = np.random.default_rng(samples)
    dt = 1e-3
    v = np.cumsum(rng.standard_normal((series, samples)), axis=1) * dt
    T = np.geomspace(0.02, 5.0, periods)
    pick = sorted({0, series // 2, series - 1})
    print("spectra case", series, samples, periods, flush=True)
    for kind in (0, 1):
        g = gpu_ctx.response_spectra(v, dt, T, 0.05, kind)
        o = oracle_lib.response_spectra(np.ascontiguousarray(v[pick]), dt, T, 0.05, kind)
        assert np.abs(o).max() > 0 and np.abs(g[pick] - o).max() <= 1e-10 * np.abs(o).max()
        one = np.array([gpu_ctx.response_spectra(v[k:k + 1], dt, T, 0.05, kind)[0] for k in pick])
        assert np.abs(g[pick] - one).max() <= 1e-12 * np.abs(o).max()


def test_records_that_are_not_finite(gpu_ctx):
    """A sample that is not a number ends the oscillator's motion, and the peak
    before it stands, also where it lies in an earlier part."""
    v = np.cumsum(np.random.default_rng(1).standard_normal((2, 900)), axis=1) * 1e-3
    T = np.geomspace(0.05, 2.0, 6)
    cut = gpu_ctx.response_spectra(np.ascontiguousarray(v[:, :300]), 1e-3, T)
    v[0, 300] = np.nan
    got = gpu_ctx.response_spectra(v, 1e-3, T)
    assert np.abs(got[0] - cut[0]).max() <= 1e-12 * cut.max() and np.all(got[1] >= cut[1] * (1 - 1e-12))
