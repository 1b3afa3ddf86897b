"""Parity of the zero-skipping weight gradient (isc_conv2d_dw) with the oracle.

Bars: |gpu - oracle| <= 1e-4 * (1 + |oracle|) elementwise against the fp64
definition; integer-valued inputs and output gradients keep every fp32
partial sum exact, so there the result equals the oracle bitwise; a zero
input gives exactly zero; two runs agree bitwise (fixed summation order).
"""
import sys

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

TOL = 1e-4


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.fixture(scope="module")
def isc(torch):
    import paper_1704_07724_amd as m
    m.lib()
    return m


def note(*parts):
    print("[case]", *parts, flush=True)
    sys.stdout.flush()


def to_dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def assert_close(got, want, what):
    got = got.astype(np.float64)
    bad = np.abs(got - want) > TOL * (1.0 + np.abs(want))
    if bad.any():
        i = np.flatnonzero(bad.ravel())[0]
        raise AssertionError("%s: %d of %d out of tolerance; first at flat %d: gpu %r oracle %r"
                             % (what, int(bad.sum()), bad.size, i, got.ravel()[i], want.ravel()[i]))


# N, C, H, W, K, R, P, sparsity: every filter size on the library's own choice of
# tile, with ragged maps and channels
DW_CASES = [
    (3, 20, 12, 12, 50, 5, 0, 0.9),     # LeNet conv2-like: 5x5, K <= 64
    (2, 7, 27, 27, 70, 5, 2, 0.9),      # AlexNet conv2-like: column tiles, ragged map group
    (2, 13, 13, 13, 64, 3, 1, 0.95),    # 3x3, one full group of maps
    (2, 23, 13, 13, 200, 3, 1, 0.9),    # 3x3, several groups of maps, ragged
    (1, 9, 20, 30, 130, 3, 1, 0.8),     # column tiles, ragged last tile
    (2, 37, 7, 7, 96, 1, 0, 0.9),       # 1x1, ragged map group
    (3, 70, 14, 14, 20, 1, 0, 0.9),     # 1x1, many channels
    (1, 2, 5, 5, 3, 5, 2, 0.5),         # tiny, filter wider than the map
    (1, 1, 1, 1, 1, 1, 0, 0.0),         # one element
]


def _dy(shape, seed):
    return np.random.default_rng(seed).standard_normal(shape).astype(np.float32)


@pytest.mark.parametrize("case", DW_CASES, ids=lambda c: "N%d-C%d-%dx%d-K%d-R%d-P%d" % c[:7])
def test_dw_matches_oracle(torch, isc, case):
    N, C, H, W, K, R, P, sp = case
    note("dw", case)
    x, _ = workloads.make_case(N, C, H, W, K, R, R, 1, P, sp, seed=41 + sum(case[:7]))
    Ho, Wo = oracle.out_size(H, R, P, 1), oracle.out_size(W, R, P, 1)
    dy = _dy((N, K, Ho, Wo), 43 + sum(case[:7]))
    got = isc.isc_conv2d_dw(to_dev(torch, x), to_dev(torch, dy), R, R, 1, P).cpu().numpy()
    want = oracle.conv2d_dw_f64(x, dy, R, R, 1, P)
    assert got.shape == want.shape
    assert_close(got, want, "dw %s" % (case,))
    # run to run: the same bits
    again = isc.isc_conv2d_dw(to_dev(torch, x), to_dev(torch, dy), R, R, 1, P).cpu().numpy()
    assert np.array_equal(got.view(np.uint32), again.view(np.uint32))


@pytest.mark.parametrize("case", DW_CASES[:7], ids=lambda c: "N%d-C%d-%dx%d-K%d-R%d-P%d" % c[:7])
def test_dw_integer_exact(torch, isc, case):
    N, C, H, W, K, R, P, sp = case
    note("dw integer", case)
    x, _ = workloads.integer_case(N, C, H, W, K, R, R, seed=47 + sum(case[:7]), sparsity=max(sp, 0.5))
    Ho, Wo = oracle.out_size(H, R, P, 1), oracle.out_size(W, R, P, 1)
    dy = np.random.default_rng(48).integers(-4, 5, (N, K, Ho, Wo)).astype(np.float32)
    got = isc.isc_conv2d_dw(to_dev(torch, x), to_dev(torch, dy), R, R, 1, P).cpu().numpy()
    assert np.array_equal(got.astype(np.float64), oracle.conv2d_dw_f64(x, dy, R, R, 1, P))


def test_dw_zero_input_and_rejects(torch, isc):
    note("dw zero input")
    x = torch.zeros((2, 5, 9, 9), device="cuda")
    dy = torch.randn((2, 6, 9, 9), device="cuda")
    dw = isc.isc_conv2d_dw(x, dy, 3, 3, 1, 1)
    assert bool((dw == 0).all()) and not bool(torch.signbit(dw).any())
    with pytest.raises(isc.IscError) as e:        # stride 2: not taken
        isc.isc_conv2d_dw(x, torch.zeros((2, 6, 5, 5), device="cuda"), 3, 3, 2, 1)
    assert e.value.status == 3
    with pytest.raises(isc.IscError) as e:        # 7x7 filter: not taken
        isc.isc_conv2d_dw(x, torch.zeros((2, 6, 9, 9), device="cuda"), 7, 7, 1, 3)
    assert e.value.status == 3


def test_dw_full_size_every_entry(torch, isc):
    """AlexNet conv2 at full size (batch 128, 96 -> 256, 27x27, 5x5, pad 2,
    sparsity 0.9) as the benchmark runs it: every entry of K x C x R x S
    against the oracle's full weight gradient."""
    layer = [l for l in workloads.WORKLOADS["alexnet_conv2"].layers][0]
    note("dw full", layer.x_shape, layer.w_shape)
    x, _ = workloads.make_inputs(layer)
    Ho = oracle.out_size(layer.H, layer.R, layer.P, 1)
    dy = _dy((layer.N, layer.K, Ho, Ho), 49)
    got = isc.isc_conv2d_dw(to_dev(torch, x), to_dev(torch, dy), layer.R, layer.S, 1, layer.P).cpu().numpy()
    want = oracle.conv2d_dw_f64(x, dy, layer.R, layer.S, 1, layer.P)
    assert_close(got, want, "dw full size")


# (N, C, H, W, K, R, P, rows, cols): every tile of the kernel, named, on maps it
# fits and on ragged ones; which tile a case runs is checked on the host
# (test_dw_plan.py)
DW_TILES = [(3, 17, 7, 7, 66, 3, 1, 7, 7), (2, 9, 5, 6, 66, 3, 1, 7, 7), (3, 9, 13, 13, 70, 3, 1, 7, 13),
            (2, 9, 10, 11, 66, 3, 1, 7, 13), (3, 9, 14, 14, 66, 3, 1, 7, 14), (2, 5, 9, 12, 66, 3, 1, 7, 14),
            (9, 9, 18, 18, 66, 3, 0, 7, 14), (2, 9, 20, 33, 66, 3, 2, 7, 14), (4, 9, 30, 29, 66, 3, 1, 4, 16),
            (3, 9, 5, 40, 66, 3, 1, 2, 16), (8, 9, 7, 7, 66, 5, 2, 7, 7), (2, 9, 4, 6, 130, 5, 2, 7, 7),
            (9, 5, 27, 27, 130, 5, 2, 9, 9), (2, 5, 10, 14, 66, 5, 1, 9, 9), (6, 5, 13, 15, 66, 5, 0, 4, 14),
            (3, 9, 11, 27, 66, 5, 2, 2, 14), (20, 35, 7, 7, 66, 1, 0, 7, 7), (8, 33, 14, 28, 66, 1, 0, 7, 14),
            (1, 33, 6, 40, 66, 1, 1, 2, 14)]


@pytest.mark.parametrize("case", DW_TILES)
def test_dw_every_tile(torch, isc, case):
    """Every compiled tile against the oracle on rectified Gaussian inputs, and
    the library's own choice within the bar of the same call."""
    N, C, H, W, K, R, P, rows, cols = case
    x, _ = workloads.make_case(N, C, H, W, K, R, R, 1, P, 0.8, seed=61 + sum(case))
    Ho, Wo = oracle.out_size(H, R, P, 1), oracle.out_size(W, R, P, 1)
    dy = _dy((N, K, Ho, Wo), 62 + sum(case))
    want = oracle.conv2d_dw_f64(x, dy, R, R, 1, P)
    for tu in ({"rows": rows, "cols": cols}, None):
        note("dw tile", case, tu)
        got = isc.isc_conv2d_dw(to_dev(torch, x), to_dev(torch, dy), R, R, 1, P, tuning=tu).cpu().numpy()
        assert_close(got, want, "dw %s %s" % (case, tu))


@pytest.mark.parametrize("case", DW_TILES)
def test_dw_tiles_and_special_values(torch, isc, case):
    """Sums of integers bitwise; and an infinite or NaN input or gradient
    reaches exactly the entries whose outputs it meets."""
    N, C, H, W, K, R, P, rows, cols = case
    tu = {"rows": rows, "cols": cols}
    note("dw tiles", case)
    rng = np.random.default_rng(sum(case))
    Ho, Wo = oracle.out_size(H, R, P, 1), oracle.out_size(W, R, P, 1)
    x, _ = workloads.integer_case(N, C, H, W, K, R, R, seed=sum(case), xmax=3)
    dy = rng.integers(-3, 4, size=(N, K, Ho, Wo)).astype(np.float32)
    got = isc.isc_conv2d_dw(to_dev(torch, x), to_dev(torch, dy), R, R, 1, P, tuning=tu).cpu().numpy()
    assert np.array_equal(got.astype(np.float64), oracle.conv2d_dw_f64(x, dy, R, R, 1, P))
    dy[dy == 0] = 1.0
    x[0, 0, H - 1, W - 1] = np.inf
    x[N - 1, C - 1, 0, 0] = np.nan
    dy[0, K - 1, Ho - 1, 0] = -np.inf
    got = isc.isc_conv2d_dw(to_dev(torch, x), to_dev(torch, dy), R, R, 1, P, tuning=tu).cpu().numpy()
    want = np.zeros((K, C, R, R))  # over the nonzero inputs only
    xp = np.pad(x.astype(np.float64), ((0, 0), (0, 0), (P, P), (P, P)))
    d = dy.astype(np.float64)
    with np.errstate(invalid="ignore"):
        for r in range(R):
            for s in range(R):
                v = xp[:, :, r:r + Ho, s:s + Wo]
                fin = np.where(np.isfinite(v), v, 0.0)
                # the finite inputs against the finite gradients, then every
                # term with an infinity or NaN on either side
                want[:, :, r, s] = np.einsum("nkij,ncij->kc", np.where(np.isfinite(d), d, 0.0), fin)
                for n, c, i, j in np.argwhere(~np.isfinite(v)):
                    want[:, c, r, s] += d[n, :, i, j] * v[n, c, i, j]
                for n, k, i, j in np.argwhere(~np.isfinite(d)):
                    nzv = np.isfinite(v[n, :, i, j]) & (v[n, :, i, j] != 0)
                    want[k, nzv, r, s] += d[n, k, i, j] * v[n, nzv, i, j]
    assert np.array_equal(got.astype(np.float64), want, equal_nan=True)


def test_dw_special_values_cost(torch, isc):
    """One NaN among AlexNet conv2's inputs costs the entries it reaches their
    range again, not all their outputs one by one: within five times the usual
    call (80 times, a thread per entry over every output)."""
    note("dw special values' cost")
    x = torch.randn((128, 96, 27, 27), device="cuda").abs_()
    x *= torch.rand_like(x) >= 0.9
    dy = torch.randn((128, 256, 27, 27), device="cuda")

    def ms(v):
        best = float("inf")
        for _ in range(4):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            isc.isc_conv2d_dw(v, dy, 5, 5, 1, 2)
            t1.record()
            t1.synchronize()
            best = min(best, t0.elapsed_time(t1))
        return best

    usual = ms(x)
    special = x.clone()
    special[100, 3, 5, 5] = float("nan")
    assert ms(special) < 5 * usual
