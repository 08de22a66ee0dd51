"""The ragged tiles of the rank-1 step: rows that are no multiple of 128 elements, at the edges of the tiling -- one strip
(up to 1024 columns) and several, rows barely longer than a block, a last strip narrower than a block, a partial last
block, fewer rows than groups, misaligned column maxima -- against the oracle, and against the general kernels."""
import numpy as np
import pytest
import torch

import oracle
import paper_2309_01507_amd as lpmm
import workloads
from gpu_util import DEV, download_state, gpu_step, run_parity, to_dev

pytestmark = pytest.mark.gpu

HP = oracle.Hyper()


@pytest.mark.parametrize("rows,cols,recipe,bf16", [
    (300, 129, "col_lognormal", False),      # shortest rows of the path: nearly every block straddles two rows
    (260, 147, "col_lognormal", True),
    (1, 129, "iid", False),                  # one whole block and one element
    (5, 1023, "iid", True),                  # one strip, few blocks
    (700, 1000, "outlier_sparse", False),    # one strip, several tiles, zero rows, scales far apart
    (9, 1025, "col_lognormal", True),        # two strips
    (67, 1030, "outlier_sparse", True),
    (40, 2049, "iid", False),                # three strips
    (33, 8193, "col_lognormal", True),       # the last strip holds one column: rows without a block in it
    (6, 8321, "col_lognormal", False),       # the last strip is one column wider than a block
    (3, 50257, "iid", True),
])
def test_step_matches_the_oracle(rows, cols, recipe, bf16):
    print(f"[gpu-test] ragged {rows}x{cols} {recipe} bf16={bf16}", flush=True)
    assert run_parity(rows, cols, steps=4, recipe=recipe, bf16=bf16, seed=71) == 0


def test_extreme_scales_take_the_exact_route():
    """Gradients around 1e-17 and 1e17: second moments beyond the reciprocal's range in some rows and columns."""
    for rows, cols in ((40, 300), (20, 1300)):
        lpmm.ensure_init(rows + cols)
        rng = np.random.default_rng(5)
        w_ref, st_ref = workloads.weights(72, 0, rows, cols).reshape(-1), oracle.state_zero(rows, cols)
        w, st = to_dev(w_ref.copy()), lpmm.new_state(rows, cols, DEV)
        for t in (1, 2, 3):
            g = rng.standard_normal((rows, cols)).astype(np.float32)
            g[: rows // 2] *= np.float32(1e-17)
            g[:, ::7] *= np.float32(1e17)
            g = g.reshape(-1)
            oracle.adamw4_step(w_ref, g, st_ref, HP, t)
            gpu_step(w, to_dev(g), st, HP, t)
            got = download_state(st)
            for x, y in ((got.m_codes, st_ref.m_codes), (got.m_scales, st_ref.m_scales), (got.v_codes, st_ref.v_codes),
                         (got.v_r, st_ref.v_r), (got.v_c, st_ref.v_c)):
                np.testing.assert_array_equal(x, y)


def test_misaligned_column_maxima():
    """Rows of whole blocks whose column maxima start 4 bytes off a 16-byte boundary: the ragged path, too."""
    rows, cols = 70, 1280
    lpmm.ensure_init(rows + cols)
    w_ref, st_ref = workloads.weights(73, 0, rows, cols).reshape(-1), oracle.state_zero(rows, cols)
    w, st = to_dev(w_ref.copy()), lpmm.new_state(rows, cols, DEV)
    st.v_colmax = torch.zeros(cols + 4, device=DEV)[1:cols + 1]
    for t in (1, 2, 3):
        g = workloads.grads(73, 0, t, rows, cols, "col_lognormal").reshape(-1)
        oracle.adamw4_step(w_ref, g, st_ref, HP, t)
        gpu_step(w, to_dev(g), st, HP, t)
    got = download_state(st)
    np.testing.assert_array_equal(got.v_codes, st_ref.v_codes)
    np.testing.assert_array_equal(got.m_codes, st_ref.m_codes)
    np.testing.assert_array_equal(got.v_c, st_ref.v_c)


@pytest.mark.parametrize("rows,cols,bf16", [(1500, 1001, False), (900, 3333, True)])
def test_same_bits_as_the_general_kernels(monkeypatch, rows, cols, bf16):
    lpmm.ensure_init(rows + cols)
    w0 = workloads.weights(74, 0, rows, cols).reshape(-1)
    grads = [workloads.grads(74, 0, t, rows, cols, "col_lognormal", bf16).reshape(-1) for t in (1, 2, 3)]
    out = []
    for general in ("0", "1"):
        monkeypatch.setenv("LPMM_FORCE_GENERAL", general)
        w, st = to_dev(w0.copy()), lpmm.new_state(rows, cols, DEV)
        for t, g in enumerate(grads, 1):
            gpu_step(w, to_dev(g, bf16), st, HP, t, bf16)
        out.append((download_state(st), w.cpu().numpy()))
    (a, wa), (b, wb) = out
    for x, y in ((a.m_codes, b.m_codes), (a.m_scales, b.m_scales), (a.v_codes, b.v_codes), (a.v_r, b.v_r), (a.v_c, b.v_c), (wa, wb)):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("rows,cols,bf16", [
    (300, 129, False),       # shortest rows of the path; the tensor's size is a multiple of 4
    (261, 147, True),        # it is not: the last row apart
    (1, 129, False),         # nothing but the last row
    (5, 1023, True),
    (258, 257, False),       # more rows than a statistics tile; the last strip holds one column
    (700, 1000, True),
    (67, 1030, False),       # two strips of the update, five of the statistics
    (33, 8193, True),
    (3, 50257, False),
])
def test_factorized_step_matches_the_oracle(rows, cols, bf16):
    from test_gpu_factor import run
    print(f"[gpu-test] ragged factorized {rows}x{cols} bf16={bf16}", flush=True)
    assert run(rows, cols, steps=3, bf16=bf16) == 0
    assert run(rows, cols, steps=2, recipe="outlier_sparse" if rows > 1 else "iid", bf16=bf16) == 0


@pytest.mark.parametrize("rows,cols,bf16", [(40, 2100, False), (67, 2305, True), (300, 777, False)])
def test_nan_in_one_second_moment_costs_that_element_only(monkeypatch, rows, cols, bf16):
    """One row's and one column's old maximum NaN, so that exactly one element's second moment is: it raises neither its
    row's nor its column's new maximum, and every state comes out as from the general kernels (rows of more than 2048
    elements; below, those record the NaN as the column's maximum).  The first moment, whose codes are searched by the
    value's bits, stays finite."""
    lpmm.ensure_init(rows + cols)
    i, j = rows // 2, cols // 3
    w0 = workloads.weights(75, 0, rows, cols).reshape(-1)
    grads = [workloads.grads(75, 0, t, rows, cols, "col_lognormal", bf16).reshape(-1) for t in (1, 2, 3)]
    out = []
    for general in ("0", "1"):
        monkeypatch.setenv("LPMM_FORCE_GENERAL", general)
        w, st = to_dev(w0.copy()), lpmm.new_state(rows, cols, DEV)
        gpu_step(w, to_dev(grads[0], bf16), st, HP, 1, bf16)
        st.v_rowmax[i] = float("nan")
        st.v_colmax[j] = float("nan")
        for t in (2, 3):
            gpu_step(w, to_dev(grads[t - 1], bf16), st, HP, t, bf16)
            if t == 2:
                first = st.v_rowmax.cpu().numpy(), st.v_colmax.cpu().numpy()
        out.append((download_state(st), w.cpu().numpy(), *first))
    (a, wa, ra, ca), (b, wb, rb, cb) = out
    assert np.isnan(wa[i * cols + j]) and np.isfinite(np.delete(wa, i * cols + j)).all()
    assert np.isfinite(ra).all() and np.isfinite(ca).all() and (ra > 0).all()
    np.testing.assert_array_equal(ra, rb)
    np.testing.assert_array_equal(a.m_codes, b.m_codes)
    np.testing.assert_array_equal(a.m_scales, b.m_scales)
    if cols > 2048:
        for x, y in ((ca, cb), (a.v_codes, b.v_codes), (a.v_r, b.v_r), (a.v_c, b.v_c), (wa, wb)):
            np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("rows,cols,plan,bf16", [(67, 8300001, False, False), (40, 16500001, False, True), (140, 4190001, True, True)])
def test_tiles_near_two_gigabytes(monkeypatch, rows, cols, plan, bf16):
    """Statistics tiles whose rows, with the one behind them, reach 2^31 bytes of fp32 elements, where the offset lies from which
    lanes without columns read: it has to stay beyond the tile.  A large gradient at that element; from a state of zeros v_t is
    (1 - beta2) g g, whose maxima are taken here by torch in the same operations."""
    monkeypatch.setenv("LPMM_FLOW", "0")
    n, hp = rows * cols, oracle.Hyper()
    lpmm.ensure_init(rows + cols)
    g = torch.rand(n, device=DEV, generator=torch.Generator(device=DEV).manual_seed(3))
    g[0x7FFFFF00 // 4] = 64.0
    if bf16:
        g = g.to(torch.bfloat16)
    w, st = torch.zeros(n, device=DEV), lpmm.new_state(rows, cols, DEV)
    h = (hp.lr, hp.beta1, hp.beta2, hp.eps, hp.weight_decay, 1)
    if plan:
        buffer = lpmm.new_plan([lpmm.make_desc(w, g, st)], 1 if bf16 else 0, DEV)
        lpmm.lpmm_adamw4_step_multi(buffer, *h)
        torch.cuda.synchronize()
        lpmm.lpmm_adamw4_plan_release(buffer)
    else:
        (lpmm.lpmm_adamw4_step_bf16g if bf16 else lpmm.lpmm_adamw4_step)(w, g, st, *h)
    row, col = [], torch.zeros(cols, device=DEV)
    omb2 = float(np.float32(1.0) - np.float32(hp.beta2))
    for x in g.view(rows, cols):
        x = x.float()
        v = (omb2 * x) * x
        row.append(v.max())
        torch.maximum(col, v, out=col)
    assert torch.equal(st.v_rowmax, torch.stack(row)) and torch.equal(st.v_colmax, col)


@pytest.mark.parametrize("rows,cols,bf16", [
    (17, 263, False),        # a row's last lane ends in the strip in front of the last one, by shift
    (25, 262, True),
    (24, 513, True),
    (9, 519, False),
    (8, 1290, True),         # tiles of 8 rows, whole
    (520, 131, True),        # several tall tiles, one strip
    (31, 2308, False),       # P = 4 (mod 8): the last 4 elements apart
    (2, 4099, True),
    (1, 4101, False),        # a single row: in parts
    (257, 129, True),        # P = 1, a tile of one row behind a whole one
    (15, 137, False),        # P = 7
    (66, 776, True),         # P = 0 (mod 8): nothing apart
])
def test_statistics_tiles_at_their_edges(rows, cols, bf16):
    """Lanes of 8 elements that start a shift into their row and end in the next one, for both forms of the second moment.  The
    maxima are exact; the sums' bound is test_gpu_factor's."""
    from test_gpu_factor import run
    print(f"[gpu-test] ragged statistics {rows}x{cols} bf16={bf16}", flush=True)
    assert run_parity(rows, cols, steps=3, recipe="col_lognormal", bf16=bf16, seed=76) == 0
    assert run(rows, cols, steps=2, bf16=bf16) == 0


@pytest.mark.parametrize("rows,cols,bf16", [(41, 2101, False), (9, 2051, True), (64, 2052, True), (264, 2049, False), (2, 2053, True)])
def test_nan_gradients_behind_the_last_whole_group(monkeypatch, rows, cols, bf16):
    """The elements behind the last multiple of 8 have the largest statistics of their columns and get NaN gradients: they raise no
    maximum, and neither does what the tiles read in their place.  As from the general kernels, which take an element at a time."""
    n, tail = rows * cols, rows * cols % 8
    lpmm.ensure_init(rows + cols)
    gen = torch.Generator(device=DEV).manual_seed(rows)
    dtype = torch.bfloat16 if bf16 else torch.float32
    g1 = (torch.rand(n, device=DEV, generator=gen) * 1e-3).to(dtype)
    g2 = torch.zeros_like(g1)
    g1[n - tail:], g2[n - tail:] = 64.0, float("nan")
    out = []
    for general in ("0", "1"):
        monkeypatch.setenv("LPMM_FORCE_GENERAL", general)
        w, st = torch.zeros(n, device=DEV), lpmm.new_state(rows, cols, DEV)
        for t, g in ((1, g1), (2, g2)):
            (lpmm.lpmm_adamw4_step_bf16g if bf16 else lpmm.lpmm_adamw4_step)(w, g, st, HP.lr, HP.beta1, HP.beta2, HP.eps, HP.weight_decay, t)
        out.append((st.v_rowmax.clone(), st.v_colmax.clone()))
    assert torch.isfinite(out[0][0]).all() and torch.isfinite(out[0][1]).all()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
