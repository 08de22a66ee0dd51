"""Stand-alone compress / decompress at the edges of their tiles: 4 elements per lane, 4096 per workgroup (with rank-1 scales 2048 in
tensors of up to 2^27), strips of 32 to 256 columns and 16 to 512 rows for the maxima; arrays at 4-byte alignment; nothing written behind a buffer's end; a NaN
costs no other element its code."""
import numpy as np
import pytest
import torch

import oracle
import paper_2309_01507_amd as lpmm
from gpu_util import DEV

pytestmark = pytest.mark.gpu

SHAPES = [(1, 3), (5, 4), (2, 63), (1100, 65), (513, 128), (31, 129), (33, 255), (67, 257), (9, 1023), (40, 1025),
          (6, 4097), (3, 8190), (4500, 7), (12, 1365)]


def _at_offset(a, dtype, words):
    """A device copy of the array that starts `words` fp32 words behind a 16-byte boundary."""
    a = np.ascontiguousarray(a).reshape(-1)
    item = a.itemsize
    buf = torch.zeros(a.size + 64, dtype=dtype, device=DEV)
    lo = words * 4 // item
    buf[lo:lo + a.size] = torch.from_numpy(a).to(DEV)
    return buf[lo:lo + a.size]


def _guarded(n, dtype, fill, words=0):
    lo = words * 4 // torch.empty(0, dtype=dtype).element_size()
    buf = torch.full((n + 64,), fill, dtype=dtype, device=DEV)
    return buf, buf[lo:lo + n], lo


def _clean(buf, lo, n, fill):
    rest = torch.cat([buf[:lo], buf[lo + n:]])
    return bool((rest == fill).all())


@pytest.mark.parametrize("rows,cols", SHAPES)
def test_compress_and_decompress_match_the_oracle(rows, cols):
    print(f"[gpu-test] convert {rows}x{cols}", flush=True)
    lpmm.ensure_init(4096)
    rng = np.random.default_rng(rows * 31 + cols)
    P, nb, half = rows * cols, (rows * cols + 127) // 128, (rows * cols + 1) // 2
    m = (rng.standard_normal((rows, cols)) * 1e-3).astype(np.float32)
    v = (rng.standard_normal((rows, cols)) ** 2 * np.exp(rng.standard_normal(cols))[None, :] * 1e-8).astype(np.float32)
    m.reshape(-1)[: min(P, 128)] = 0.0
    v[rows // 2, :] = 0.0
    v[:, cols // 2] = 0.0
    if P > 200:
        v.reshape(-1)[200:] *= np.float32(1e-35)            # scales outside the reciprocal's range
    want = {0: oracle.quant_m(m), 1: oracle.quant_v(v), 2: oracle.quant_v_block(v)}
    sizes = {0: (nb, 0), 1: (rows, cols), 2: (nb, 0)}
    for which, x in ((0, m), (1, v), (2, v)):
        for words in (0, 1, 3):
            xin = _at_offset(x, torch.float32, words)
            cb, codes, clo = _guarded(half, torch.uint8, 0xEE, words)
            na, nb_ = sizes[which]
            ab, sa, alo = _guarded(na, torch.float32, -1.0, words)
            bb, sb, blo = _guarded(nb_, torch.float32, -1.0, words) if nb_ else (None, None, 0)
            lpmm.lpmm_quant_state(which, xin, rows, cols, codes, sa, sb)
            ob, out, olo = _guarded(P, torch.float32, -7.0, words)
            lpmm.lpmm_dequant_state(which, codes, sa, sb, rows, cols, out)
            torch.cuda.synchronize()
            w = want[which]
            np.testing.assert_array_equal(sa.cpu().numpy(), w[1])
            np.testing.assert_array_equal(codes.cpu().numpy(), w[0])
            assert _clean(cb, clo, half, 0xEE) and _clean(ab, alo, na, -1.0) and _clean(ob, olo, P, -7.0)
            if which == 1:
                np.testing.assert_array_equal(sb.cpu().numpy(), w[2])
                assert _clean(bb, blo, nb_, -1.0)
                dec = oracle.dequant_v(w[0], w[1], w[2]).reshape(-1)
            else:
                dec = (oracle.dequant_m if which == 0 else oracle.dequant_v_block)(w[0], w[1], P)
            np.testing.assert_array_equal(out.cpu().numpy(), dec)


@pytest.mark.parametrize("what", ["state", "b128/de", "b2048/de", "b128/de signed", "b2048/de0 stochastic"])
def test_nan_raises_no_block_scale(what):
    """NaNs in a block, a whole lane's 4 elements among them: scales and all other codes as with zeros in their place.
    (The block-wise second moment and the ablation quantizers: they search no table by the value's bits.)"""
    lpmm.ensure_init(4096)
    rows, cols = 9, 1000
    P = rows * cols
    rng = np.random.default_rng(17)
    x = (rng.standard_normal((rows, cols)) * np.exp(rng.standard_normal((rows, cols)))).astype(np.float32)
    if "signed" not in what:
        x = np.abs(x)
    bad = np.zeros(P, bool)
    for lo, n in ((0, 4), (132, 4), (257, 1), (700, 12), (2048, 8), (4099, 5), (P - 4, 4)):
        bad[lo:lo + n] = True
    bad = bad.reshape(rows, cols)
    clean = np.where(bad, np.float32(0.0), x)
    dirty = torch.from_numpy(np.where(bad, np.float32("nan"), x)).to(DEV).reshape(-1)
    codes = torch.full(((P + 1) // 2,), 0xEE, dtype=torch.uint8, device=DEV)
    if what == "state":
        want_codes, want_scales = oracle.quant_v_block(clean)
        sa = torch.full((want_scales.size,), -1.0, device=DEV)
        lpmm.lpmm_quant_state(2, dirty, rows, cols, codes, sa, None)
    else:
        norm, map_name = what.split()[0].split("/")
        signed, stochastic = "signed" in what, "stochastic" in what
        want_codes, want_scales, _ = oracle.quant_ablation(clean, norm, map_name, signed, stochastic, 5)
        sa = torch.full((want_scales.size,), -1.0, device=DEV)
        lpmm.lpmm_quant_ablation(lpmm.NORM_B128 if norm == "b128" else lpmm.NORM_B2048,
                                 lpmm.MAP_DE if map_name == "de" else lpmm.MAP_DE0, signed, int(stochastic), 5, dirty, rows,
                                 cols, codes, sa, None)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(sa.cpu().numpy(), want_scales)
    got, want = (oracle.unpack_codes(c, P) for c in (codes.cpu().numpy(), want_codes))
    np.testing.assert_array_equal(got[~bad.reshape(-1)], want[~bad.reshape(-1)])
    assert (got[bad.reshape(-1)] == 0).all()


@pytest.mark.parametrize("rows,cols", [(1, 1), (16, 8), (17, 9), (33, 128), (31, 136), (65, 264), (300, 519), (5, 2049), (12289, 129), (800001, 3)])
def test_maxima_at_the_edges_of_their_tiles(rows, cols):
    """Lanes repeat the last 8 columns and rows the last one; 4 to 16 lanes a row up to 128 columns, 32 beyond; 16 to 512 rows a tile."""
    print(f"[gpu-test] maxima {rows}x{cols}", flush=True)
    lpmm.ensure_init(4096)
    gen = torch.Generator(device=DEV).manual_seed(rows + cols)
    v = torch.rand(rows, cols, generator=gen, device=DEV)
    v[torch.rand(rows, cols, generator=gen, device=DEV) < 0.01] = float("nan")
    v[torch.rand(rows, cols, generator=gen, device=DEV) < 0.01] = -0.0
    v[rows // 2] = -1.0
    v[:, cols // 3] *= -1.0
    v[-1, -1], v[0, 0] = 3.0, 2.0
    z = torch.where(v > 0, v, torch.zeros_like(v))
    for words in (0, 1):
        buf = torch.empty(rows * cols + 8, device=DEV)
        x = buf[words:words + rows * cols]
        x.copy_(v.reshape(-1))
        codes = torch.zeros((rows * cols + 7) // 8 * 4, dtype=torch.uint8, device=DEV)[:(rows * cols + 1) // 2]
        r, c = torch.full((rows + 1,), -5.0, device=DEV), torch.full((cols + 1,), -5.0, device=DEV)
        lpmm.lpmm_quant_state(1, x, rows, cols, codes, r[:rows], c[:cols])
        assert torch.equal(r[:rows], z.amax(1)) and torch.equal(c[:cols], z.amax(0))
        assert r[rows] == -5.0 and c[cols] == -5.0


@pytest.mark.parametrize("rows,cols", [(1, 150001), (3, 600007), (8, 300000), (33, 90001), (64, 100003), (70, 200001), (200, 83001),    # runs of strips
                                       (1, 5), (4, 3), (70001, 7), (5000, 9), (4097, 15), (3001, 33), (513, 63),             # one at a time
                                       (5000, 8), (4097, 12), (3001, 32), (2049, 36), (1025, 64), (1025, 65)])
def test_maxima_of_few_rows_and_of_few_columns(rows, cols):
    """In rows of more than 82000 elements a workgroup takes several strips, and stores the columns' maxima where it has all rows; 4, 8, 16 or 32 lanes a
    row, up to 64 columns an element at a time where rows begin anywhere."""
    print(f"[gpu-test] maxima {rows}x{cols}", flush=True)
    lpmm.ensure_init(4096)
    gen = torch.Generator(device=DEV).manual_seed(rows + cols)
    v = torch.rand(rows, cols, generator=gen, device=DEV) - 0.5 / min(rows, cols)
    v[torch.rand(rows, cols, generator=gen, device=DEV) < 0.01] = float("nan")
    z = torch.where(v > 0, v, torch.zeros_like(v))
    for words in (0, 1):
        buf = torch.empty(rows * cols + 8, device=DEV)
        x = buf[words:words + rows * cols]
        x.copy_(v.reshape(-1))
        codes = torch.zeros((rows * cols + 7) // 8 * 4, dtype=torch.uint8, device=DEV)[:(rows * cols + 1) // 2]
        r, c = torch.full((rows + 1,), -5.0, device=DEV), torch.full((cols + 1,), -5.0, device=DEV)
        lpmm.lpmm_quant_state(1, x, rows, cols, codes, r[:rows], c[:cols])
        assert torch.equal(r[:rows], z.amax(1)) and torch.equal(c[:cols], z.amax(0))
        assert r[rows] == -5.0 and c[cols] == -5.0


def test_a_single_long_row_takes_no_queue_of_atomics():
    """One row of 10^7 elements against a square of as many: 100 us and 27; 480 with an atomic on the row's maximum per 256 columns."""
    lpmm.ensure_init(1 << 22)
    n = 3162 * 3162
    x = torch.rand(n, device=DEV)
    codes, scales = torch.zeros((n + 7) // 8 * 4, dtype=torch.uint8, device=DEV)[:n // 2], torch.zeros(n + 1, device=DEV)

    def best(rows, cols):
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                lpmm.lpmm_quant_state(1, x, rows, cols, codes, scales[cols:cols + rows], scales[:cols])
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times[1:])

    row, square = best(1, n), best(3162, 3162)
    assert row < 8 * square, (row, square)


@pytest.mark.parametrize("rows,cols", [(3, 683), (2, 1025), (16384, 8192), (16385, 8193)])
def test_second_moment_in_short_and_long_workgroups(rows, cols):
    """Two runs of 1024 elements a workgroup up to 2^27 elements, four beyond.  Against the definitions in fp32: decompressed values
    exactly, codes but for values within rounding of a boundary (two roundings of 2^-24 in 16 n, boundaries 1 apart: below 1e-6 of them)."""
    print(f"[gpu-test] second moment {rows}x{cols}", flush=True)
    lpmm.ensure_init(4096)
    gen = torch.Generator(device=DEV).manual_seed(cols)
    v = torch.rand(rows, cols, generator=gen, device=DEV)
    n = rows * cols
    codes = torch.zeros((n + 7) // 8 * 4, dtype=torch.uint8, device=DEV)[:(n + 1) // 2]
    r, c, out = torch.zeros(rows, device=DEV), torch.zeros(cols, device=DEV), torch.full((n + 1,), -5.0, device=DEV)
    lpmm.lpmm_quant_state(1, v, rows, cols, codes, r, c)
    lpmm.lpmm_dequant_state(1, codes, r, c, rows, cols, out[:n])
    q = torch.stack((codes & 15, codes >> 4), 1).reshape(-1)[:n].view(rows, cols).float()
    scale = torch.minimum(r[:, None], c[None, :])
    assert torch.equal(out[:n].view(rows, cols), (q + 1) * 0.0625 * scale) and out[n] == -5.0
    want = torch.clamp(torch.ceil(16 * (v / scale) - 1.5), 0, 15)
    assert int((want != q).sum()) <= 1e-6 * n
