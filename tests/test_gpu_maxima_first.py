"""The rank-1 step takes the maxima of the new second moment first and updates everything afterwards.  Edges of both passes'
tiles against the oracle: half-empty strips (an odd number of column blocks), super-tiles cut off by the last row, rows that
lie 32 KiB apart and rows that do not, one and two rows per group, more workgroups than one ticket line, the ragged tiles'
straddling blocks, left-over last rows and partial last blocks; extreme scales, which send whole tiles down the exact route."""
import numpy as np
import pytest
import torch

import oracle
import paper_2309_01507_amd as lpmm
import workloads
from gpu_util import DEV, PARAM_ATOL, PARAM_RTOL, download_state, gpu_step, to_dev

pytestmark = pytest.mark.gpu
HP = oracle.Hyper()

SHAPES = [(1, 128), (7, 128), (9, 384), (513, 256), (520, 640), (65, 1024), (200, 1024), (17, 4096), (40, 8192), (24, 1152),
          (33, 9216), (300, 1792),                                     # whole blocks per row
          (1, 130), (3, 129), (67, 257), (129, 1023), (50, 1025), (21, 2305), (5, 8191), (1000, 131)]      # ragged


def _check(rows, cols, bf16, scale=1.0, steps=3, seed=5):
    lpmm.ensure_init(rows + cols)
    w_ref = workloads.weights(seed, 0, rows, cols).reshape(-1)
    st_ref = oracle.state_zero(rows, cols)
    w, st = to_dev(w_ref.copy()), lpmm.new_state(rows, cols, DEV)
    for t in range(1, steps + 1):
        g = workloads.grads(seed, 0, t, rows, cols, "outlier_sparse").reshape(-1) * np.float32(scale)
        gd = to_dev(g, bf16)
        g = gd.float().cpu().numpy()
        oracle.adamw4_step(w_ref, g, st_ref, HP, t)
        gpu_step(w, gd, st, HP, t, bf16)
        torch.cuda.synchronize()
        got = download_state(st)
        tag = "%d x %d bf16=%s scale=%g step %d" % (rows, cols, bf16, scale, t)
        for name in ("m_scales", "v_r", "v_c", "m_codes", "v_codes"):
            np.testing.assert_array_equal(getattr(got, name), getattr(st_ref, name), err_msg=tag + " " + name)
        np.testing.assert_allclose(w.cpu().numpy(), w_ref, rtol=PARAM_RTOL, atol=PARAM_ATOL, err_msg=tag)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("rows,cols", SHAPES)
def test_tile_edges(rows, cols, bf16):
    _check(rows, cols, bf16)


@pytest.mark.parametrize("rows,cols,bf16", [(131333, 128, False), (66000, 256, True), (2900, 3072, True)])
def test_tall_and_narrow(rows, cols, bf16):
    """Tiles of 64 rows in the second pass, up to 512 rows in the first; 3 workgroups of the second pass per CU."""
    _check(rows, cols, bf16, steps=2)


@pytest.mark.parametrize("rows,cols", [(40, 1152), (70, 257)])
def test_extreme_scales(rows, cols):
    """Second moments around 2^-120: scales below 2^-100, which neither a reciprocal nor a sixteenth keeps whole."""
    _check(rows, cols, False, scale=1e-14)


@pytest.mark.parametrize("env", [{"LPMM_GX": "1"}, {"LPMM_GX": "3"}, {"LPMM_RW": "64"}, {"LPMM_RS": "5"}, {"LPMM_RW2": "512"},
                                 {"LPMM_RW2": "9"}])
def test_tilings(monkeypatch, env):
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    _check(300, 1792, True)
    _check(520, 1024, False)
