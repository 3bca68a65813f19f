"""GPU parity: thanos_factor against the CPU oracle."""
import numpy as np
import pytest

from oracle import thanos_oracle as orc
from synth import LayerSpec, make_calibration

pytestmark = pytest.mark.gpu


def _h(b, T=None, rho=0.7, seed=0, outliers=False):
    X = make_calibration(LayerSpec("t", c=1, b=b, tokens=T or 4 * b, dtype="f16", rho=rho,
                                   k_mix=8, seed=seed, outliers=outliers))
    return orc.hessian(X).astype(np.float32)


@pytest.mark.parametrize("b", [128, 200, 512, 640, 1000, 1408, 2432])
def test_factor_matches_oracle(b):
    from tests.gpu_util import gpu_factor
    print(f"factor b={b}", flush=True)
    H32 = _h(b, seed=b)
    U, xn2, info = gpu_factor(H32, 0.01)
    assert info == 0
    np.testing.assert_array_equal(xn2, np.diag(H32))
    assert np.all(np.tril(U, -1) == 0.0)
    Hd = orc.damped(H32.astype(np.float64), 0.01)
    Uref = orc.inverse_factor(Hd)
    U64 = U.astype(np.float64)
    # fp32 factorisation: error ~ cond(scaled H_d) * 2^-24; these inputs have cond ~ 1e3
    assert np.linalg.norm(U64 - Uref) <= 2e-4 * np.linalg.norm(Uref)
    # defining property, independent of the oracle's route: U^T U H_d = I
    R = U64.T @ (U64 @ Hd) - np.eye(b)
    assert np.max(np.abs(R)) < 5e-3
    # every residual inverse (what Alg. 1 recomputes per block) is contained in U
    for j in (0, b // 3, b - 5):
        inv = np.linalg.inv(Hd[j:, j:])
        got = U64[j:, j:].T @ U64[j:, j:]
        assert np.linalg.norm(got - inv) <= 5e-4 * np.linalg.norm(inv)


def test_factor_heavy_tailed_channels():
    from tests.gpu_util import gpu_factor
    H32 = _h(640, seed=9, outliers=True)
    U, _, info = gpu_factor(H32, 0.01)
    assert info == 0
    Uref = orc.inverse_factor(orc.damped(H32.astype(np.float64), 0.01))
    assert np.linalg.norm(U - Uref) <= 5e-4 * np.linalg.norm(Uref)


def test_not_positive_definite_is_reported():
    from tests.gpu_util import gpu_factor
    H32 = _h(256, seed=1)
    H32[100, 100] = -1.0
    _, _, info = gpu_factor(H32, 0.0)
    assert info > 0


@pytest.mark.parametrize("b", [1, 31, 33, 97, 129, 2944, 3200, 4096, 4100])
def test_factor_tile_edges(b):
    """One block that is mostly padding, 32-tiles cut at their edges, and the sizes around which the factorisation
    passes from one launch per step to two-level updates in front of such steps (32 blocks of 128)."""
    from tests.gpu_util import gpu_factor
    H32 = _h(b, T=2 * b + 64, seed=b)
    U, _, info = gpu_factor(H32, 0.01)
    assert info == 0
    assert np.all(np.tril(U, -1) == 0.0)
    Uref = orc.inverse_factor(orc.damped(H32.astype(np.float64), 0.01))
    # condition numbers of some thousands at 2 b tokens: some 1e3 * 2^-24, as in the test above
    assert np.linalg.norm(U - Uref) <= 2e-4 * np.linalg.norm(Uref)


@pytest.mark.parametrize("col", [0, 1, 4, 5, 31, 32, 70, 127, 128, 200])
def test_first_bad_pivot_is_named(col):
    """The elimination runs from the last column backwards: the first pivot that fails is that of the
    one negative entry of a diagonal matrix, wherever it sits in its pair, tile and block."""
    from tests.gpu_util import gpu_factor
    H32 = np.diag(np.linspace(1.0, 2.0, 256)).astype(np.float32)
    H32[col, col] = -1.0
    _, _, info = gpu_factor(H32, 0.0)
    assert info == col + 1


@pytest.mark.parametrize("b,lo,hi", [(200, 40, 40), (200, -40, -40), (712, -40, -40), (300, -36, 36)])
def test_powers_of_two_scale_exactly(b, lo, hi):
    """H -> D H D with powers of two d_j (undamped): U -> U D^-1 bit for bit, for scales at which the
    product of two pivots leaves the range of fp32, equal in all channels and mixed."""
    from tests.gpu_util import gpu_factor
    H32 = _h(b, seed=5)
    g = np.random.default_rng(b)
    d = np.ldexp(np.float32(1.0), g.integers(lo, hi + 1, size=b))
    U1, _, i1 = gpu_factor(H32, 0.0)
    U2, xn2, i2 = gpu_factor((H32 * d[:, None] * d[None, :]).astype(np.float32), 0.0)
    assert i1 == i2 == 0
    np.testing.assert_array_equal(xn2, np.diag(H32) * d * d)
    np.testing.assert_array_equal(U2 * d[None, :], U1)


@pytest.mark.parametrize("b", [700, 3200])
def test_split_products_ranges(b):
    """The products that split their operands into two 16-bit values: merges of the inverse (700) and
    wide updates too (3200), on channels whose scales span 2^+-20 and of which every fourth is nearly
    the copy of its neighbour, so that the inverse of the scaled factor grows to about 2^6.  Powers of
    two still scale exactly, and the error stays that of an fp32 factorisation: the condition number
    of the scaled matrix is about b + 2^13 (one unit in 2^12 of a channel is its own), times 2^-24
    and 8 for the walk of the sums."""
    from tests.gpu_util import gpu_factor
    g = np.random.default_rng(b)
    X = g.standard_normal((2 * b, b))
    k = b // 4
    X[:, 1:4 * k:4] = X[:, 0:4 * k:4] + 2.0 ** -6 * g.standard_normal((2 * b, k))
    H32 = (X.T @ X).astype(np.float32)
    d = np.ldexp(np.float32(1.0), g.integers(-20, 21, size=b))
    U1, _, i1 = gpu_factor(H32, 0.0)
    U2, _, i2 = gpu_factor((H32 * d[:, None] * d[None, :]).astype(np.float32), 0.0)
    assert i1 == i2 == 0
    np.testing.assert_array_equal(U2 * d[None, :], U1)
    Uref = orc.inverse_factor(H32.astype(np.float64))
    assert np.abs(Uref).max() * np.sqrt(2 * b) > 2.0 ** 5
    assert np.linalg.norm(U1 - Uref) <= 8 * (b + 2.0 ** 13) * 2.0 ** -24 * np.linalg.norm(Uref)


@pytest.mark.parametrize("b", [128, 256, 300, 512, 1365, 3200, 4096, 4100])
def test_well_conditioned_factor_is_as_exact_as_fp32(b):
    """H = D (I + E) D with eigenvalues of I + E between 1/2 and 3/2: no condition number hides the products'
    own errors.  The values right of the diagonal of U D are, relative to their column, within 2^-20 of float64 (sums of up
    to 512 values at a time, each rounded at 2^-24; measured 3.3 to 4.6e-7), in the root mean square over the columns:
    operands of 18 bits or fewer, or a split that loses its remainder in some tile, would show."""
    from tests.gpu_util import gpu_factor
    g = np.random.default_rng(b)
    E = np.triu(g.standard_normal((b, b)) * (0.25 / np.sqrt(b)), 1)
    d = np.exp(g.standard_normal(b))
    H32 = ((np.eye(b) + E + E.T) * d[:, None] * d[None, :]).astype(np.float32)
    U, _, info = gpu_factor(H32, 0.0)
    assert info == 0
    Uref = orc.inverse_factor(H32.astype(np.float64)) * np.sqrt(np.diag(H32).astype(np.float64))[None, :]
    err = np.triu(U * np.sqrt(np.diag(H32).astype(np.float64))[None, :] - Uref, 1)
    rel = np.linalg.norm(err[:, 8:], axis=0) / np.linalg.norm(np.triu(Uref, 1)[:, 8:], axis=0)
    rms = float(np.sqrt(np.mean(rel * rel)))
    print(f"b={b}: rms {rms:.2e}, worst column {rel.max():.2e}", flush=True)
    assert rms <= 2.0 ** -20
