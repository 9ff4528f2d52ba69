"""Projections of many rows to feature counts that no workgroup tile divides, against the oracle: every tile with its last one
partly used (by 16 features up to all but 16), ragged rows, split outputs, and the memory past the outputs untouched."""
import numpy as np
import pytest
import torch

from oracle import model_ref as R
from test_gpu_model import M, check_close, dev, draw, host  # noqa: F401  (M is the fixture)

pytestmark = pytest.mark.gpu


def guarded(rows, N):
    """A [rows][N] output with a row of a known pattern behind it."""
    buf = torch.full((rows + 1, N), 7.0, dtype=torch.bfloat16, device="cuda")
    return buf, buf[:rows]


@pytest.mark.parametrize("rows,K,N,tile", [(640, 96, 208, (64, 64, 2)), (130, 160, 1040, (64, 64, 2)), (130, 32, 12320, (128, 128, 2)),
                                           (1000, 64, 4112, (128, 256, 1)), (1000, 96, 8208, (256, 256, 1)),
                                           (2000, 32, 8208, (128, 128, 1)), (257, 4096, 1968, (64, 64, 2))])
def test_linear(M, rows, K, N, tile):
    x, w, res = draw(1, (rows, K)), draw(2, (N, K), K ** -0.5), draw(3, (rows, N))
    ref = R.linear(x, w, res)
    mass = np.abs(R.bf16_to_f64(x)) @ np.abs(R.bf16_to_f64(w)).T
    pw = M.bctm_pack_weight(dev(w))
    assert M.bctm_linear_tile(rows, K, N, tiled=True) == tile
    bits = []
    for xin in (M.bctm_pack_rows(dev(x)), dev(x)):
        buf, out = guarded(rows, N)
        M.bctm_linear(xin, pw, dev(res), out)
        check_close(host(out), ref, 2.0 ** -20 * mass, f"linear {rows}x{K}x{N}")
        assert bool((buf[rows] == 7.0).all())
        bits.append(host(out))
    assert np.array_equal(*bits)


@pytest.mark.parametrize("rows,K,N,tile", [(128, 96, 2080, (64, 32, 2)), (128, 96, 6176, (128, 32, 2)), (130, 32, 6176, (128, 64, 2)), (150, 64, 12320, (128, 128, 1)),
                                           (300, 32, 12320, (256, 128, 1)), (520, 32, 12320, (128, 256, 1)),
                                           (700, 32, 12320, (128, 64, 1)), (1030, 1024, 160, (64, 32, 2))])
def test_swiglu(M, rows, K, N, tile):
    x, wg, wu = draw(5, (rows, K)), draw(6, (N, K), 2.0 * K ** -0.5), draw(7, (N, K), K ** -0.5)
    xa = np.abs(R.bf16_to_f64(x))
    g, u = R.linear_f64(x, wg), R.linear_f64(x, wu)
    mg, mu = xa @ np.abs(R.bf16_to_f64(wg)).T, xa @ np.abs(R.bf16_to_f64(wu)).T
    slack = 2.0 ** -20 * (1.1 * mg * np.abs(u) + (np.abs(g) + 1.0) * mu + np.abs(g * u))
    pg, pu, xt = M.bctm_pack_weight(dev(wg)), M.bctm_pack_weight(dev(wu)), M.bctm_pack_rows(dev(x))
    assert M.bctm_linear_tile(rows, K, N, swiglu=True, tiled=True) == tile
    buf, out = guarded(rows, N)
    M.bctm_swiglu(xt, pg, pu, out)
    check_close(host(out), R.swiglu(x, wg, wu), slack, f"swiglu {rows}x{K}x{N}")
    assert bool((buf[rows] == 7.0).all())
    tiled = M.bctm_swiglu(xt, pg, pu, tiled=True)   # the same values in the tiled order
    again = M.bctm_pack_rows(out)
    whole = rows // 32 * 32 * N * 2
    assert torch.equal(tiled.data.view(-1).view(torch.uint8)[:whole], again.data.view(-1).view(torch.uint8)[:whole])


def test_split_outputs(M):
    rows, K, widths = 300, 192, (1008, 144, 528)   # 1680 features: borders and the end inside tiles
    x = draw(1, (rows, K))
    ws = [draw(20 + i, (n, K), K ** -0.5) for i, n in enumerate(widths)]
    bufs, outs = zip(*[guarded(rows, n) for n in widths])
    assert M.bctm_linear_plan(rows, K, sum(widths)) == M.BCTM_KERNEL_TILE128
    M.bctm_linear_split(M.bctm_pack_rows(dev(x)), M.bctm_pack_weight(*[dev(a) for a in ws]), outs)
    for b, o, wi in zip(bufs, outs, ws):
        m = np.abs(R.bf16_to_f64(x)) @ np.abs(R.bf16_to_f64(wi)).T
        check_close(host(o), R.linear(x, wi, None), 2.0 ** -20 * m, "split")
        assert bool((b[rows] == 7.0).all())
