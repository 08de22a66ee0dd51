"""The ablation quantizers of the second moment on the GPU (lpmm_quant_ablation / lpmm_dequant_ablation: Sec. 4.1,
Tab. 1, stochastic rounding of App. D.3) against the oracle: codes, scales and decompressed values bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2309_01507_amd as lpmm
from gpu_util import DEV, to_dev

pytestmark = pytest.mark.gpu

NORM = {"b128": lpmm.NORM_B128, "b2048": lpmm.NORM_B2048, "rank1": lpmm.NORM_RANK1}
MAP = {"de": lpmm.MAP_DE, "de0": lpmm.MAP_DE0, "linear": lpmm.MAP_LINEAR}
# every quantizer of Tab. 1 (second moment), the signed ones of its first line (first moment), and the rest of the grid
COMBOS = [(n, m, False) for n in ("b2048", "b128", "rank1") for m in ("de", "de0", "linear")] + \
         [("b2048", "de", True), ("b128", "de", True)]


def _input(rows, cols, signed, seed):
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal((rows, cols)) * np.exp(2 * rng.standard_normal((rows, cols)))).astype(np.float32)
    if not signed:
        x = (x * x).astype(np.float32)
    if rows > 4:
        x[3, :] = 0.0                                 # a zero row
    flat = x.reshape(-1)
    if flat.size > 4096:
        flat[2048:4096] = 0.0                         # a zero block of 2048 (and 16 of 128)
    return x


def _gpu_quant(x, norm, map_name, signed, stochastic, seed):
    rows, cols = x.shape
    na, nb = lpmm.ablation_scale_sizes(NORM[norm], rows, cols)
    codes = torch.full((((x.size + 1) // 2 + 3) // 4 * 4,), 0xEE, dtype=torch.uint8, device=DEV)[:(x.size + 1) // 2]
    sa = torch.full((na,), -1.0, device=DEV)
    sb = torch.full((max(nb, 1),), -1.0, device=DEV)
    lpmm.lpmm_quant_ablation(NORM[norm], MAP[map_name], signed, int(stochastic), seed, to_dev(x.reshape(-1)), rows, cols,
                             codes, sa, sb if nb else None)
    return codes, sa, sb


@pytest.mark.parametrize("norm,map_name,signed", COMBOS)
@pytest.mark.parametrize("shape", [(21, 300), (64, 2048), (1, 130), (257, 1031)])
@pytest.mark.parametrize("stochastic", [False, True])
def test_ablation_quantizers_match_the_oracle(norm, map_name, signed, shape, stochastic):
    rows, cols = shape
    print(f"[gpu-test] ablation {norm}/{map_name} signed={signed} sr={stochastic} {rows}x{cols}", flush=True)
    lpmm.ensure_init(4096)
    x = _input(rows, cols, signed, seed=rows * 7 + cols)
    seed = 1234567 + rows
    want_codes, want_sa, want_sb = oracle.quant_ablation(x, norm, map_name, signed, stochastic, seed)
    codes, sa, sb = _gpu_quant(x, norm, map_name, signed, stochastic, seed)
    torch.cuda.synchronize()
    P = x.size
    got = oracle.unpack_codes(codes.cpu().numpy(), P)
    np.testing.assert_array_equal(sa.cpu().numpy(), want_sa, err_msg="scale_a")
    if norm == "rank1":
        np.testing.assert_array_equal(sb.cpu().numpy(), want_sb, err_msg="scale_b")
    np.testing.assert_array_equal(got, oracle.unpack_codes(want_codes, P), err_msg="codes")
    if P % 2:
        assert int(codes[-1]) >> 4 == 0                               # the unused nibble of an odd tail stays 0
    out = torch.full((P,), -7.0, device=DEV)
    lpmm.lpmm_dequant_ablation(NORM[norm], MAP[map_name], signed, codes, sa, sb if norm == "rank1" else None, rows, cols, out)
    want = oracle.dequant_ablation(want_codes, want_sa, want_sb, rows, cols, norm, map_name, signed)
    np.testing.assert_array_equal(out.cpu().numpy().reshape(rows, cols), want)


@pytest.mark.parametrize("norm", ["b128", "b2048"])
@pytest.mark.parametrize("shape", [(1, 2048), (1, 2049), (3, 1365), (2048, 1024), (2048, 1025)])
def test_stochastic_rounding_in_short_and_long_workgroups(norm, shape):
    """Up to 2^21 elements a workgroup takes one block of 2048 with stochastic rounding, beyond two."""
    x = _input(*shape, False, seed=shape[0] + shape[1])
    want_codes, want_sa, _ = oracle.quant_ablation(x, norm, "de", False, True, 99)
    codes, sa, _ = _gpu_quant(x, norm, "de", False, True, 99)
    np.testing.assert_array_equal(sa.cpu().numpy(), want_sa)
    np.testing.assert_array_equal(oracle.unpack_codes(codes.cpu().numpy(), x.size), oracle.unpack_codes(want_codes, x.size))


def test_stochastic_rounding_depends_on_the_seed_only():
    """Same seed, same codes, whatever was launched before; another seed, other codes; each code is the nearest
    entry or its neighbour."""
    lpmm.ensure_init(4096)
    x = _input(300, 1024, False, seed=5)
    a = _gpu_quant(x, "b128", "de", False, True, 11)[0].clone()
    _gpu_quant(_input(64, 256, False, seed=6), "rank1", "de0", False, True, 12)
    b = _gpu_quant(x, "b128", "de", False, True, 11)[0]
    c = _gpu_quant(x, "b128", "de", False, True, 13)[0]
    near = _gpu_quant(x, "b128", "de", False, False, 0)[0]
    assert torch.equal(a, b) and not torch.equal(a, c)
    ua, un = oracle.unpack_codes(a.cpu().numpy(), x.size).astype(int), oracle.unpack_codes(near.cpu().numpy(), x.size).astype(int)
    assert np.abs(ua - un).max() == 1


def test_bad_arguments_are_refused():
    import ctypes
    lpmm.ensure_init(4096)
    L = lpmm.lib()
    t = torch.zeros(4096, device=DEV)
    p = t.data_ptr()
    shape = (ctypes.c_int64 * 2)(4, 128)
    q = lambda *a: L.lpmm_quant_ablation(*a, 0, p, ctypes.addressof(shape), p, p, p, None)
    assert q(2, 0, 1, 0) == -1          # rank-1 of signed input
    assert q(0, 1, 1, 0) == -1          # signed DE-0
    assert q(3, 0, 0, 0) == -1          # no such normalization
    assert q(0, 0, 0, 2) == -1          # no such rounding
    assert L.lpmm_quant_ablation(2, 0, 0, 0, 0, p, ctypes.addressof(shape), p, p, None, None) == -1     # rank-1 without column maxima
    assert L.lpmm_dequant_ablation(0, 5, 0, p, p, None, ctypes.addressof(shape), p, None) == -1
    torch.cuda.synchronize()


@pytest.mark.parametrize("norm,map_name,signed", COMBOS)
@pytest.mark.parametrize("stochastic", [False, True])
def test_values_around_entries_and_thresholds(norm, map_name, signed, stochastic):
    """Normalized values on, and a few units in the last place around, every entry and decision threshold, under scales that are
    and are not powers of two, tiny and huge ones and zero; for rank-1, under row maxima that hold for the row alone."""
    T = lpmm.lpmm_ablation_table(MAP[map_name], signed).astype(np.float64)
    at = np.concatenate([T, (T[1:] + T[:-1]) / 2, [0.0]]).astype(np.float32)
    n = np.concatenate([at] + [np.nextafter(at, np.float32(s), dtype=np.float32) for s in (-4, 4)] +
                       [at * np.float32(1 + k * 2.0 ** -22) for k in (-9, -3, 3, 9)])
    n = n[(np.abs(n) <= 1) & ((n >= 0) | signed)]
    rng = np.random.default_rng(17)
    rows = []
    for s in (1.0, 0.37, 3.1e-7, 1.9999999, 2.0 ** -99.5, 1.7e29, 1e-33, 3e38, 0.0):
        x = rng.choice(n, 4096) * np.float32(s)
        x[::128] = s                                    # every block, of either size, and every row and column block holds its scale
        rows.append(x.astype(np.float32))
    x = np.stack(rows)
    if norm == "rank1":
        x[:, 1::2] = np.where(x[:, 1::2] > 0, x[:, 1::2], 0)
    want_codes, want_sa, want_sb = oracle.quant_ablation(x, norm, map_name, signed, stochastic, 4711)
    codes, sa, sb = _gpu_quant(x, norm, map_name, signed, stochastic, 4711)
    np.testing.assert_array_equal(sa.cpu().numpy(), want_sa)
    if norm == "rank1":
        np.testing.assert_array_equal(sb.cpu().numpy(), want_sb)
    np.testing.assert_array_equal(oracle.unpack_codes(codes.cpu().numpy(), x.size), oracle.unpack_codes(want_codes, x.size))


@pytest.mark.parametrize("stochastic", [False, True])
@pytest.mark.parametrize("shape", [(3, 683), (2048, 1024), (2048, 1025)])
def test_rank1_in_short_and_long_workgroups(shape, stochastic):
    """Up to 2^21 elements a workgroup takes two runs of 1024, beyond four."""
    x = _input(*shape, False, seed=shape[0] + shape[1])
    want_codes, want_sa, want_sb = oracle.quant_ablation(x, "rank1", "de0", False, stochastic, 99)
    codes, sa, sb = _gpu_quant(x, "rank1", "de0", False, stochastic, 99)
    np.testing.assert_array_equal(sa.cpu().numpy(), want_sa)
    np.testing.assert_array_equal(sb.cpu().numpy(), want_sb)
    np.testing.assert_array_equal(oracle.unpack_codes(codes.cpu().numpy(), x.size), oracle.unpack_codes(want_codes, x.size))


@pytest.mark.parametrize("norm,map_name,signed", COMBOS)
def test_stochastic_rounding_of_zeros_and_values_next_to_zero(norm, map_name, signed):
    """Zeros of both signs, values down to the smallest subnormal ones, values a few units in the last place from an entry and NaN
    among ordinary ones, under scales that let n = x / s underflow and such that do not: 2^21 elements, so that random numbers next to
    0 and 1 (64 within 2^-16) meet all of them."""
    print(f"[gpu-test] ablation next to zero {norm}/{map_name} signed={signed}", flush=True)
    rng = np.random.default_rng(23)
    T = lpmm.lpmm_ablation_table(MAP[map_name], signed)
    rows, cols = 1024, 2048
    n = np.exp2(-150 * rng.random((rows, cols))).astype(np.float32)
    kind = rng.integers(0, 5, (rows, cols))
    n[kind == 0] = 0
    near = rng.choice(T, (rows, cols)) * (1 + rng.integers(-6, 7, (rows, cols)) * np.float32(2.0 ** -23))
    n = np.where(kind == 1, np.minimum(near, 1), n).astype(np.float32)
    n[kind == 2] = rng.random(int((kind == 2).sum()), dtype=np.float32)
    if signed:
        n = np.where(rng.random((rows, cols)) < 0.5, -n, n)
    n[(kind == 0) & (rng.random((rows, cols)) < 0.5)] = -0.0
    x = n * np.exp2(rng.integers(-90, 91, (rows, 1))).astype(np.float32)
    if not signed:
        x = np.maximum(x, np.float32(-0.0))
    x[rng.random((rows, cols)) < 0.001] = np.nan
    want_codes, want_sa, want_sb = oracle.quant_ablation(x, norm, map_name, signed, True, 4712)
    codes, sa, sb = _gpu_quant(x, norm, map_name, signed, True, 4712)
    np.testing.assert_array_equal(sa.cpu().numpy(), want_sa)
    if norm == "rank1":
        np.testing.assert_array_equal(sb.cpu().numpy(), want_sb)
    np.testing.assert_array_equal(oracle.unpack_codes(codes.cpu().numpy(), x.size), oracle.unpack_codes(want_codes, x.size))


@pytest.mark.parametrize("signed", [False, True])
def test_zeros_cost_stochastic_rounding_no_second_route(signed):
    """A value that is 0, or small against its scale, takes no longer than another: half of them zeros 30 us as without any, 48 where
    every wave with one did its elements twice.  The best of several runs of 20, so that other work on the machine does not count."""
    rows, cols = 4096, 4096
    gen = torch.Generator(device=DEV).manual_seed(3)
    dense = torch.rand(rows, cols, generator=gen, device=DEV) + 0.01
    if signed:
        dense *= torch.where(torch.rand(rows, cols, generator=gen, device=DEV) < 0.5, -1.0, 1.0)
    half = torch.where(torch.rand(rows, cols, generator=gen, device=DEV) < 0.5, dense, torch.zeros_like(dense))
    small = dense * torch.where(torch.rand(rows, cols, generator=gen, device=DEV) < 0.5, 1.0, 1e-9)
    codes, sa = torch.zeros(rows * cols // 2, dtype=torch.uint8, device=DEV), torch.zeros(rows * cols // 128, device=DEV)

    def best(x):
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                lpmm.lpmm_quant_ablation(lpmm.NORM_B128, lpmm.MAP_DE, signed, lpmm.ROUND_STOCHASTIC, 7, x, rows, cols, codes, sa, None)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times[1:])

    lpmm.ensure_init(4096)
    t = {name: best(x) for name, x in (("dense", dense), ("half", half), ("small", small), ("dense again", dense))}
    assert max(t["half"], t["small"]) < 1.25 * max(t["dense"], t["dense again"]), t


@pytest.mark.parametrize("norm,map_name,signed", COMBOS)
@pytest.mark.parametrize("stochastic", [False, True])
def test_runs_of_zeros(norm, map_name, signed, stochastic):
    """Waves of nothing but zeros, of either sign, inside blocks and rows with other values and in ones without, at a tensor's end too."""
    rng = np.random.default_rng(29)
    x = rng.random((37, 1001)).astype(np.float32)
    if signed:
        x *= rng.choice(np.float32([-1, 1]), x.shape)
    flat = x.reshape(-1)
    for first in range(0, flat.size, 2048):
        k = first + int(rng.integers(0, 1024))
        flat[k:k + int(rng.integers(200, 1500))] = rng.choice(np.float32([0.0, -0.0]))
    x[5:9], flat[-700:] = 0.0, 0.0
    x[:, 300:310] = 0.0
    want_codes, want_sa, want_sb = oracle.quant_ablation(x, norm, map_name, signed, stochastic, 4713)
    codes, sa, sb = _gpu_quant(x, norm, map_name, signed, stochastic, 4713)
    np.testing.assert_array_equal(sa.cpu().numpy(), want_sa)
    if norm == "rank1":
        np.testing.assert_array_equal(sb.cpu().numpy(), want_sb)
    np.testing.assert_array_equal(oracle.unpack_codes(codes.cpu().numpy(), x.size), oracle.unpack_codes(want_codes, x.size))
