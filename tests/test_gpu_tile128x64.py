"""Projections in tiles of 128 rows x 64 columns with K in two parts, and bands of 1 to 7 row tiles, against the oracle: one K
step (the second part has none), odd and even counts, ragged rows and feature counts, in place on the residual."""
import numpy as np
import pytest

from oracle import model_ref as R
from test_gpu_model import M, check_close, dev, draw, host  # noqa: F401  (M is the fixture)
from test_gpu_ragged_widths import guarded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,K,N", [(129, 32, 6144), (200, 64, 6208), (255, 288, 6144), (600, 96, 3264), (770, 224, 2304),
                                      (850, 160, 2288), (1000, 96, 2048), (1100, 128, 1792), (1408, 320, 1472)])
def test_linear(M, rows, K, N):
    x, w, res = draw(1, (rows, K)), draw(2, (N, K), K ** -0.5), draw(3, (rows, N))
    pw = M.bctm_pack_weight(dev(w))
    assert M.bctm_linear_tile(rows, K, N, tiled=True) == M.bctm_linear_tile(rows, K, N) == (128, 64, 2)
    mass = np.abs(R.bf16_to_f64(x)) @ np.abs(R.bf16_to_f64(w)).T
    ref, bits = R.linear(x, w, res), []
    for xin in (M.bctm_pack_rows(dev(x)), dev(x)):
        buf, out = guarded(rows, N)
        out.copy_(dev(res))
        M.bctm_linear(xin, pw, out, out)
        check_close(host(out), ref, 2.0 ** -20 * mass, f"linear {rows}x{K}x{N}")
        assert bool((buf[rows] == 7.0).all())
        bits.append(host(out))
    assert np.array_equal(*bits)


@pytest.mark.parametrize("rows,K,N", [(129, 32, 3072), (600, 96, 1616), (850, 160, 1152)])
def test_swiglu(M, rows, K, N):
    x, wg, wu = draw(5, (rows, K)), draw(6, (N, K), 2.0 * K ** -0.5), draw(7, (N, K), K ** -0.5)
    assert M.bctm_linear_tile(rows, K, N, swiglu=True, tiled=True) == (128, 32, 2)
    xa = np.abs(R.bf16_to_f64(x))
    g, u = R.linear_f64(x, wg), R.linear_f64(x, wu)
    mg, mu = xa @ np.abs(R.bf16_to_f64(wg)).T, xa @ np.abs(R.bf16_to_f64(wu)).T
    slack = 2.0 ** -20 * (1.1 * mg * np.abs(u) + (np.abs(g) + 1.0) * mu + np.abs(g * u))
    buf, out = guarded(rows, N)
    M.bctm_swiglu(M.bctm_pack_rows(dev(x)), M.bctm_pack_weight(dev(wg)), M.bctm_pack_weight(dev(wu)), out)
    check_close(host(out), R.swiglu(x, wg, wu), slack, f"swiglu {rows}x{K}x{N}")
    assert bool((buf[rows] == 7.0).all())
