"""GPU parity: thanos_prune_layer against the CPU oracle.

Bar: masks bit-exact on inputs without near-ties; W_hat within 1e-3 relative Frobenius error;
reconstruction error within 1 % of the oracle's.  Both sides receive the same fp32 Hessian, so
the first block's selection is taken on identical numbers on both sides; later blocks see
weights that differ by fp32 rounding, which can only flip decisions whose margin is at that
level (checked through the margins the oracle reports).
"""
import numpy as np
import pytest

from oracle import thanos_oracle as orc
from synth import LayerSpec, make_weight, make_calibration

pytestmark = pytest.mark.gpu


def _layer(c, b, T, dtype="f32", rho=0.7, seed=0, outliers=False):
    spec = LayerSpec("t", c=c, b=b, tokens=T, dtype=dtype, rho=rho, k_mix=16, seed=seed,
                     outliers=outliers)
    W = make_weight(spec)
    X = make_calibration(spec)
    H32 = orc.hessian(X).astype(np.float32)
    return W, H32


def _rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


def _check(W, H32, Wg, Mg, Wo, Mo, exact_mask=True):
    H = H32.astype(np.float64)
    if exact_mask:
        np.testing.assert_array_equal(Mg, Mo)
    assert np.all(Wg[Mg == 1] == 0.0)
    if np.array_equal(Mg, Mo):
        assert _rel(Wg, Wo) < 1e-3
    eo = orc.reconstruction_error(W, Wo, H)
    eg = orc.reconstruction_error(W, Wg.astype(np.float64), H)
    assert abs(eg - eo) <= 0.01 * eo + 1e-12


# --------------------------------------------------------------------------- configuration 1
@pytest.mark.parametrize("rho", [0.0, 0.7])
def test_cfg1_unstructured(rho):
    from tests.gpu_util import gpu_prune
    # seeds searched on the CPU so that the oracle's smallest decision margin is > 5e-6
    W, H32 = _layer(512, 512, 2048, "f32", rho=rho, seed={0.0: 0, 0.7: 4}[rho])
    print(f"cfg1 unstructured rho={rho}", flush=True)
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=0.5, B=128)
    assert info == 0
    assert int(Mg.sum()) == 512 * 512 // 2
    Wo, Mo, margins = orc.prune_unstructured(W, H32.astype(np.float64), 0.5, 128, 0.01,
                                             return_margins=True)
    assert margins.min() > 5e-6, "seed has a near-tie; pick another"
    _check(W, H32, Wg, Mg, Wo, Mo)
    # the same decisions when the oracle ranks the plain float64 metric instead of the one rounded
    # to float32 like the kernel's: with margins > 5e-6 a rounding of ~2e-7 decides nothing
    _, Mo64 = orc.prune_unstructured(W, H32.astype(np.float64), 0.5, 128, 0.01,
                                     metric_dtype=np.float64)
    np.testing.assert_array_equal(Mg, Mo64)
    Wm, _ = orc.magnitude_prune(W, p=0.5)
    H = H32.astype(np.float64)
    assert orc.reconstruction_error(W, Wg.astype(np.float64), H) <= orc.reconstruction_error(W, Wm, H)


@pytest.mark.parametrize("n,m,rho", [(2, 4, 0.0), (2, 4, 0.7), (4, 8, 0.7), (1, 4, 0.7), (3, 4, 0.7)])
def test_cfg1_nm(n, m, rho):
    from tests.gpu_util import gpu_prune
    W, H32 = _layer(512, 512, 2048, "f32", rho=rho, seed=1)
    print(f"cfg1 {n}:{m} rho={rho}", flush=True)
    Wg, Mg, info = gpu_prune(W, H32, mode="nm", n=n, m=m, B=128)
    assert info == 0
    assert np.all(Mg.reshape(512, 512 // m, m).sum(axis=2) == n)
    Wo, Mo, mg = orc.prune_nm(W, H32.astype(np.float64), n, m, 128, 0.01, return_margins=True)
    bad_rows = np.unique(np.nonzero(Mg != Mo)[0])
    # a differing group must be a near-tie in the oracle (fp32 vs fp64 weights after updates)
    if len(bad_rows):
        gi, gj = np.nonzero((Mg != Mo).reshape(512, 512 // m, m).any(axis=2))
        first = {}
        for i, j in zip(gi, gj):
            first.setdefault(i, j)
        for i, j in first.items():
            assert mg[i, j] < 1e-4, (i, j, mg[i, j])
        assert len(bad_rows) <= 2
    print(f"  rows whose mask differs from the free-running oracle: {len(bad_rows)}", flush=True)
    # every decision of every block (not only the first differing one of a row) against the
    # oracle's decision on the weights that block saw; W_hat and reconstruction error per row
    from tests.fullsize_util import check_nm_rows
    Hd64 = H32.astype(np.float64)
    check_nm_rows(W, Hd64, orc.inverse_factor(orc.damped(Hd64, 0.01)), Wg.astype(np.float64), Mg,
                  n, m, 128, 0.01, f"cfg1 {n}:{m} rho={rho}")
    ok = np.setdiff1d(np.arange(512), bad_rows)
    np.testing.assert_array_equal(Mg[ok], Mo[ok])
    assert _rel(Wg[ok], Wo[ok]) < 1e-3
    _check(W, H32, Wg, Mg, Wo, Mo, exact_mask=False)
    # oracle ranking the plain float64 metric: same masks wherever its own margins are clear
    _, Mo64, mg64 = orc.prune_nm(W, H32.astype(np.float64), n, m, 128, 0.01,
                                 metric_dtype=np.float64, return_margins=True)
    clear = np.all(mg64 > 1e-5, axis=1)
    assert clear.mean() > 0.95
    np.testing.assert_array_equal(Mg[clear & np.isin(np.arange(512), ok)],
                                  Mo64[clear & np.isin(np.arange(512), ok)])


# --------------------------------------------------------------------------- ragged shapes
@pytest.mark.parametrize("c,b,B,mode", [
    (100, 328, 128, "unstructured"),    # c not a multiple of anything, last block 72 wide
    (100, 328, 128, "nm"),
    (67, 200, 64, "unstructured"),      # one column per lane
    (67, 200, 32, "nm"),
    (130, 260, 100, "unstructured"),    # B not a power of two
    (50, 150, 50, "unstructured"),      # B and b not multiples of 4: scalar load paths
    (96, 768, 256, "unstructured"),     # block size 256 (configuration 5), 4 wavefronts per row
    (64, 640, 256, "nm"),               # last block 128 wide
    (40, 450, 200, "unstructured"),     # wide block, nothing aligned
    (9, 40, 128, "unstructured"),       # single narrow block
    (5, 16, 1, "unstructured"),         # B = 1
    (70, 1216, 512, "nm"),              # block 512 (the n:m setting of the Experiments section): 256 unknowns per row,
                                        # last block 192 wide
    (48, 768, 256, "nm14"),             # 1:4 at block 256: 64 unknowns per row in a wide block
    # b not a multiple of 8 at more than toy size: the scalar / 8-byte paths of the sweep
    (300, 1100, 128, "unstructured"),   # b % 8 == 4
    (300, 1100, 128, "nm"),
    (257, 1030, 128, "unstructured"),   # b % 4 == 2: nothing 16-byte aligned from row to row
    # large blocks of the block-size ablation: more than 256 unknowns per row, tile grids in
    # global memory, workgroups that walk the rows
    (40, 2304, 1024, "nm"),             # 512 unknowns per row; last block 256 wide (LDS path)
    (30, 1100, 512, "unstructured"),    # up to 512 unknowns, ragged last block of 76
    (600, 1536, 1024, "nm"),            # more rows than resident workgroups
    (24, 4608, 2048, "nm"),             # 1024 unknowns per row
    (16, 4096, 4096, "nm14"),           # one block of 4096 columns, 1024 unknowns per row
    # rows that lose more than half of a block are solved through the inverse of the block's G
    # (complement form: bw - s unknowns)
    (32, 1024, 512, "nm34"),            # 3:4: 384 removed per row and block -> 128 unknowns
    (20, 2048, 1024, "unstructured"),   # up to 512 unknowns either way: tile grids in global memory
    (48, 1024, 256, "unstructured70"),  # 70 %: most rows go the complement way, some do not
])
def test_ragged_shapes(c, b, B, mode):
    from tests.gpu_util import gpu_prune
    W, H32 = _layer(c, b, 4 * b, "f32", seed=c + b)
    print(f"ragged c={c} b={b} B={B} {mode}", flush=True)
    H = H32.astype(np.float64)
    from tests.fullsize_util import check_nm_rows, check_unstructured_rows
    if mode.startswith("unstructured"):
        p = 0.7 if mode.endswith("70") else 0.5
        Wg, Mg, info, tau = gpu_prune(W, H32, mode="unstructured", p=p, B=B, tau=True)
        Wo, Mo = orc.prune_unstructured(W, H, p, B, 0.01)
        assert int(Mg.sum()) == orc.num_to_remove(p, c, b)
    else:
        n, m = {"nm14": (1, 4), "nm34": (3, 4)}.get(mode, (2, 4))
        Wg, Mg, info = gpu_prune(W, H32, mode="nm", n=n, m=m, B=B)
        Wo, Mo = orc.prune_nm(W, H, n, m, B, 0.01)
    assert info == 0
    if np.array_equal(Mg, Mo):
        _check(W, H32, Wg, Mg, Wo, Mo)
        return
    # the masks differ: every differing decision must be a near-tie of the oracle on the weights
    # the block saw, and W_hat must match the oracle under the GPU's mask row by row
    print(f"  masks differ at {int((Mg != Mo).sum())} positions: checking decision by decision",
          flush=True)
    assert (Mg != Mo).mean() < 1e-3
    U = orc.inverse_factor(orc.damped(H, 0.01))
    if mode.startswith("unstructured"):
        check_unstructured_rows(W, H, U, Wg.astype(np.float64), Mg, tau, p, B, 0.01, f"ragged {c}x{b}")
    else:
        check_nm_rows(W, H, U, Wg.astype(np.float64), Mg, n, m, B, 0.01, f"ragged {c}x{b}")


def test_cfg5_like_block256_heavy_tailed():
    # configuration 5 in small: N(0, 0.015^2) fp16 weights, outlier channels, 60 % unstructured,
    # block 256
    from tests.gpu_util import gpu_prune
    spec = LayerSpec("t", c=160, b=1024, tokens=4096, dtype="f16", w_std=0.015, rho=0.7, k_mix=16,
                     seed=11, outliers=True)
    W, X = make_weight(spec), make_calibration(spec)
    H32 = orc.hessian(X).astype(np.float32)
    H = H32.astype(np.float64)
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=0.6, B=256)
    assert info == 0
    assert int(Mg.sum()) == orc.num_to_remove(0.6, 160, 1024)
    Wo, Mo = orc.prune_fast(W, H, mode="unstructured", p=0.6, B=256, damp=0.01)
    assert (Mg != Mo).mean() < 1e-4
    Wt, _ = orc.prune_fast(W, H, mode="unstructured", p=0.6, B=256, damp=0.01, mask_in=Mg)
    assert _rel(Wg, Wt) < 1e-3
    eo = orc.reconstruction_error(W, Wo, H)
    eg = orc.reconstruction_error(W, Wg.astype(np.float64), H)
    assert abs(eg - eo) <= 0.01 * eo
    # 4:8 at block 256: s = 128 per row
    Wg, Mg, info = gpu_prune(W, H32, mode="nm", n=4, m=8, B=256)
    assert info == 0
    assert np.all(Mg.reshape(160, 128, 8).sum(axis=2) == 4)
    Wt, _ = orc.prune_fast(W, H, mode="nm", n=4, m=8, B=256, damp=0.01, mask_in=Mg)
    assert _rel(Wg, Wt) < 1e-3
    _, Mo = orc.prune_fast(W, H, mode="nm", n=4, m=8, B=256, damp=0.01)
    assert (Mg != Mo).mean() < 1e-3


# --------------------------------------------------------------------------- outlier rows
@pytest.mark.parametrize("alpha,n,m,B,use_factor", [(0.1, 2, 4, 128, False), (0.25, 4, 8, 64, True)])
def test_nm_with_outlier_rows(alpha, n, m, B, use_factor):
    """n:m algorithm with alpha > 0 (App. G.4.4): the ceil(alpha c) rows of largest loss
    h_i = W_i H W_i^T stay dense and untouched, the others are pruned as usual."""
    from tests.gpu_util import gpu_factor, gpu_prune
    c, b = 200, 384
    W, H32 = _layer(c, b, 2048, "f16", rho=0.7, seed=21)
    # spread the row norms: the ranking of the row losses is then decided far above fp32 noise
    scale = np.linspace(0.5, 2.0, c)[np.random.default_rng(5).permutation(c)]
    W = (W.astype(np.float64) * scale[:, None]).astype(np.float16)
    H = H32.astype(np.float64)
    n_out = orc.num_outlier_rows(alpha, c)
    h = np.sort(orc.row_losses(W.astype(np.float64), H))
    assert (h[c - n_out] - h[c - n_out - 1]) / h[c - n_out] > 1e-3   # margin at the cut
    rows = orc.pruned_rows(W.astype(np.float64), H, alpha)
    print(f"outlier rows alpha={alpha} {n}:{m} B={B}", flush=True)
    kw = {}
    if use_factor:   # H is still needed for the row losses
        U, xn2, info = gpu_factor(H32, 0.01)
        assert info == 0
        kw = dict(U=U, xnorm2=xn2)
    Wg, Mg, info = gpu_prune(W, H32, mode="nm", n=n, m=m, B=B, alpha=alpha, **kw)
    assert info == 0
    # outlier rows: untouched, no mask
    np.testing.assert_array_equal(Mg[~rows], 0)
    np.testing.assert_array_equal(Wg[~rows], W[~rows].astype(np.float32))
    assert (~rows).sum() == n_out
    # pruned rows: exact n:m pattern, parity with the oracle
    assert np.all(Mg[rows].reshape(rows.sum(), b // m, m).sum(axis=2) == n)
    Wo, Mo, mg = orc.prune_nm(W, H, n, m, B, 0.01, return_margins=True, alpha=alpha)
    diff_rows = np.unique(np.nonzero(Mg != Mo)[0])
    for i in diff_rows:   # a differing group must be a near-tie in the oracle
        j = np.nonzero((Mg[i] != Mo[i]).reshape(b // m, m).any(axis=1))[0][0]
        assert mg[i, j] < 1e-4, (i, j, mg[i, j])
    assert len(diff_rows) <= 2
    ok = np.setdiff1d(np.arange(c), diff_rows)
    assert _rel(Wg[ok], Wo[ok]) < 1e-3
    Wt, _ = orc.prune_fast(W, H, mode="nm", n=n, m=m, B=B, damp=0.01, mask_in=Mg)
    assert _rel(Wg, Wt) < 1e-3


def test_outlier_rows_argument_checks():
    import torch
    import paper_2504_05346_amd as th
    o = th.PruneOpts(mode=th.THANOS_UNSTRUCTURED, sparsity=0.5, block_size=128, damping=0.01,
                     outlier_fraction=0.1)
    assert th.thanos_prune_workspace_bytes(64, 128, o) == 0          # not defined for Alg. 1
    o = th.PruneOpts(mode=th.THANOS_NM, n=2, m=4, block_size=128, damping=0.01,
                     outlier_fraction=1.0)
    assert th.thanos_prune_workspace_bytes(64, 128, o) == 0          # alpha must be < 1
    o0 = th.PruneOpts(mode=th.THANOS_NM, n=2, m=4, block_size=128, damping=0.01)
    o1 = th.PruneOpts(mode=th.THANOS_NM, n=2, m=4, block_size=128, damping=0.01,
                      outlier_fraction=0.1)
    assert th.thanos_prune_workspace_bytes(64, 128, o1) > th.thanos_prune_workspace_bytes(64, 128, o0)


# --------------------------------------------------------------------------- structured (Alg. 2)
@pytest.mark.parametrize("c,b,p,alpha,dtype", [(200, 384, 0.5, 0.0, "f16"), (150, 300, 0.3, 0.1, "f32"),
                                               (64, 1000, 0.25, 0.2, "f16"),
                                               (1536, 2048, 0.25, 0.05, "f16")])   # several tiles each way
def test_structured(c, b, p, alpha, dtype):
    """Alg. 2: s = ceil(p b / (1 - alpha)) columns of smallest loss removed from the
    non-outlier rows in one shot."""
    from tests.gpu_util import gpu_prune
    W, H32 = _layer(c, b, 4 * b, dtype, rho=0.7, seed=31)
    rng = np.random.default_rng(9)
    W = (W.astype(np.float64) * np.linspace(0.5, 2.0, c)[rng.permutation(c)][:, None]
         * np.linspace(0.6, 1.8, b)[rng.permutation(b)][None, :]).astype(W.dtype)
    H = H32.astype(np.float64)
    s = orc.num_columns_to_remove(p, alpha, b)
    rows = orc.pruned_rows(W.astype(np.float64), H, alpha)
    v = np.sort(orc.column_losses(W.astype(np.float64), np.diag(H), rows))
    assert (v[s] - v[s - 1]) / v[s] > 1e-4            # margin at the column cut
    print(f"structured {c}x{b} p={p} alpha={alpha}", flush=True)
    Wg, Mg, info = gpu_prune(W, H32, mode="structured", p=p, alpha=alpha, cast=True)[:3]
    assert info == 0
    Wo, Mo = orc.prune_structured(W, H, p, alpha, 0.01)
    np.testing.assert_array_equal(Mg, Mo)
    assert np.all(Wg[Mg == 1] == 0.0)
    np.testing.assert_array_equal(Wg[~rows], W[~rows].astype(np.float32))
    assert _rel(Wg, Wo) < 1e-3
    eo = orc.reconstruction_error(W, Wo, H)
    eg = orc.reconstruction_error(W, Wg.astype(np.float64), H)
    assert abs(eg - eo) <= 0.01 * eo


def test_structured_argument_checks():
    import paper_2504_05346_amd as th
    ok = th.PruneOpts(mode=th.THANOS_STRUCTURED, sparsity=0.5, damping=0.01, outlier_fraction=0.1)
    assert th.thanos_prune_workspace_bytes(64, 128, ok) > 0
    bad = th.PruneOpts(mode=th.THANOS_STRUCTURED, sparsity=0.8, damping=0.01, outlier_fraction=0.5)
    assert th.thanos_prune_workspace_bytes(64, 128, bad) == 0        # p / (1 - alpha) > 1


# --------------------------------------------------------------------------- forced masks
def test_given_mask_with_empty_and_full_rows():
    from tests.gpu_util import gpu_prune
    c, b, B = 96, 384, 128
    W, H32 = _layer(c, b, 2048, "f32", seed=5)
    g = np.random.default_rng(0)
    M = (g.random((c, b)) < g.random((c, 1))).astype(np.uint8)   # per-row density 0..1
    M[0] = 0
    M[1] = 1
    M[2, :128] = 1
    M[3, 128:256] = 0
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=0.5, B=B, mask_in=M)
    assert info == 0
    np.testing.assert_array_equal(Mg, M)
    Wo, Mo = orc.prune_fast(W, H32.astype(np.float64), mode="unstructured", p=0.5, B=B, damp=0.01,
                            mask_in=M)
    assert np.all(Wg[M == 1] == 0.0)
    np.testing.assert_array_equal(Wg[0], W[0])           # nothing removed: row untouched
    assert np.all(Wg[1] == 0.0)
    assert _rel(Wg, Wo) < 1e-3
    rows = np.linalg.norm(Wg - Wo, axis=1) / np.maximum(np.linalg.norm(Wo, axis=1), 1e-30)
    assert rows.max() < 1e-3


@pytest.mark.parametrize("given_factor", [False, True])  # with: every row direct, without: complement above half
@pytest.mark.parametrize("B", [256, 200])
def test_given_mask_with_every_tile_count(B, given_factor):
    """Blocks wider than 128 columns: systems at the edges of the 32-column tiles, 0 to B unknowns."""
    from tests.gpu_util import gpu_prune, gpu_factor
    b = 2 * B
    sizes = [s for t in range(0, B + 1, 32) for s in (t - 1, t, t + 1) if 0 <= s <= B] + [B - 1, B]
    c = len(sizes)
    W, H32 = _layer(c, b, 4 * b, "f32", seed=B)
    g = np.random.default_rng(B)
    M = np.zeros((c, b), np.uint8)
    for i, s in enumerate(sizes):
        M[i, g.permutation(B)[:s]] = 1
        M[i, B + g.permutation(B)[:sizes[-1 - i]]] = 1
    kw = {}
    if given_factor:
        U, xn2, info = gpu_factor(H32, 0.01)
        assert info == 0
        kw = dict(U=U, xnorm2=xn2)
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=0.5, B=B, mask_in=M, **kw)
    assert info == 0
    np.testing.assert_array_equal(Mg, M)
    Wo, _ = orc.prune_fast(W, H32.astype(np.float64), mode="unstructured", p=0.5, B=B, damp=0.01,
                           mask_in=M)
    assert np.all(Wg[M == 1] == 0.0)
    # fp32 solves of systems with condition numbers of some hundreds: errors of a few 1e-5 (the
    # other parity tests of this file allow the same 1e-3)
    rows = np.linalg.norm(Wg - Wo, axis=1) / np.maximum(np.linalg.norm(Wo, axis=1), 1e-30)
    assert rows.max() < 1e-3


@pytest.mark.parametrize("c,b,B", [
    (2048, 256, 128),   # all rows at once in the kernel for 96 unknowns
    (2049, 253, 128),   # 64 unknowns and complement; last block of 125 columns
    (4096, 200, 128),   # last block of 72
    (4097, 242, 97),    # five rows to a workgroup; odd blocks, the last of 48
    (5120, 128, 128),   # the last number of rows with five
    (5121, 189, 128),   # four again; last block of 61
])
def test_given_mask_with_every_row_size_up_to_128_columns(c, b, B):
    """Rows of 0 to B unknowns in a block of up to 128 columns, for the numbers of rows at which the solver changes.
    Rows are independent: the first ones, which have every size, and the last ones are checked."""
    from tests.gpu_util import gpu_prune
    W, H32 = _layer(c, b, 4 * b, "f32", seed=c)
    print(f"row sizes {c}x{b} B={B}", flush=True)
    g = np.random.default_rng(c)
    M = np.zeros((c, b), np.uint8)
    for j in range(0, b, B):
        w = min(B, b - j)
        first = np.argsort(g.random((c, w)), axis=1).argsort(axis=1)
        M[:, j:j + w] = first < ((np.arange(c) + j) % (w + 1))[:, None]
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=0.5, B=B, mask_in=M)
    assert info == 0
    np.testing.assert_array_equal(Mg, M)
    assert np.all(Wg[M == 1] == 0.0)
    at = np.unique(np.concatenate([np.arange(2 * B + 2), np.arange(c - 16, c)]))
    Wo, _ = orc.prune_fast(W[at], H32.astype(np.float64), mode="unstructured", p=0.5, B=B, damp=0.01, mask_in=M[at])
    # of the row that came in: what is left of one that loses all but a weight or two is a difference of values of that size
    rows = np.linalg.norm(Wg[at] - Wo, axis=1) / np.linalg.norm(W[at], axis=1)
    # two systems of the condition number of the scaled matrix (50 to 80), the factor and the row, each at 2^-24; products
    # of operands without their lower halves, 11 bits, are off by hundreds of times as much
    Hd = orc.damped(H32.astype(np.float64), 0.01)
    kappa = np.linalg.cond(Hd / np.sqrt(np.outer(np.diag(Hd), np.diag(Hd))))
    print(f"worst row {rows.max():.2e}, allowed {2 * kappa * 2.0 ** -24:.2e}", flush=True)
    assert rows.max() < 2 * kappa * 2.0 ** -24


def test_factor_reuse_matches_internal_factor():
    from tests.gpu_util import gpu_prune, gpu_factor
    W, H32 = _layer(64, 256, 1024, "f32", seed=6)
    U, xn2, info = gpu_factor(H32, 0.01)
    a = gpu_prune(W, H32, mode="nm", n=2, m=4, B=128)
    b_ = gpu_prune(W, None, mode="nm", n=2, m=4, B=128, U=U, xnorm2=xn2)
    np.testing.assert_array_equal(a[1], b_[1])
    np.testing.assert_array_equal(a[0], b_[0])


@pytest.mark.parametrize("c,b,B,p", [
    (2560, 768, 256, 0.6),    # whole row tiles, last block whole
    (2603, 700, 256, 0.75),   # ragged rows, last block 188 wide
    (2570, 836, 512, 0.5),    # up to 256 unknowns, rows on either side of half a block
])
def test_complement_form_for_many_rows(c, b, B, p):
    """From 2560 rows on the complement's products with K run as matrix products over all rows."""
    from tests.gpu_util import gpu_prune
    W, H32 = _layer(c, b, 4 * b, "f32", seed=c)
    W[:3] *= 1e-3     # loses whole blocks
    W[3:6] *= 1e3     # loses next to nothing
    H = H32.astype(np.float64)
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=p, B=B)
    assert info == 0
    assert int(Mg.sum()) == orc.num_to_remove(p, c, b)
    assert np.all(Wg[Mg == 1] == 0.0)
    Wo, _ = orc.prune_fast(W, H, mode="unstructured", p=p, B=B, damp=0.01, mask_in=Mg)
    some = np.linalg.norm(Wo, axis=1) > 0
    rows = np.linalg.norm(Wg - Wo, axis=1)[some] / np.linalg.norm(Wo, axis=1)[some]
    assert rows.max() < 1e-3  # as in the other parity tests of this file
    _, Mo = orc.prune_fast(W, H, mode="unstructured", p=p, B=B, damp=0.01)
    assert (Mo != Mg).mean() < 1e-4


def test_complement_form_for_more_row_tiles_than_run_at_once():
    """The products that turn the complement's results into multipliers have two column tiles per row
    tile, and here 548 of them for 512 places: whole blocks on both sides of the alternating multiplier
    buffers, and a last one of four columns.  Rows of a given mask are independent: some are checked."""
    from tests.gpu_util import gpu_prune
    c, b, B, p = 35000, 772, 256, 0.6
    W, H32 = _layer(c, b, 4 * b, "f32", seed=12)
    print(f"many row tiles {c}x{b}", flush=True)
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=p, B=B)
    assert info == 0
    assert int(Mg.sum()) == orc.num_to_remove(p, c, b)
    assert np.all(Wg[Mg == 1] == 0.0)
    at = np.unique(np.concatenate([np.arange(0, c, 97), np.arange(c - 128, c)]))
    Wo, _ = orc.prune_fast(W[at], H32.astype(np.float64), mode="unstructured", p=p, B=B, damp=0.01,
                           mask_in=Mg[at])
    rows = np.linalg.norm(Wg[at] - Wo, axis=1) / np.maximum(np.linalg.norm(Wo, axis=1), 1e-30)
    assert rows.max() < 1e-3  # as in the other parity tests of this file


# --------------------------------------------------------------------------- ties
@pytest.mark.parametrize("B", [64, 128, 256])   # one block size per per-row solver
def test_exact_ties_follow_row_major_order(B):
    # Diagonal Hessian: no surviving weight moves, so every block sees heavily tied metrics
    # (weights from a 5-value set); the mask must equal one global psi with (row, col) ties.
    from tests.gpu_util import gpu_prune
    g = np.random.default_rng(1)
    c, b = 40, 512
    W = g.choice(np.array([-2.0, -1.0, 0.5, 1.0, 2.0], dtype=np.float32), size=(c, b))
    H32 = np.diag(g.choice(np.array([1.0, 4.0], dtype=np.float32), size=b))
    for p in (0.5, 0.3):
        print(f"ties B={B} p={p}", flush=True)
        Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=p, B=B, damp=0.01)
        assert info == 0
        Mref = orc.psi(W, np.diag(H32), orc.num_to_remove(p, c, b))
        np.testing.assert_array_equal(Mg, Mref)
        np.testing.assert_array_equal(Wg, W * (1 - Mref))
    Wg, Mg, _ = gpu_prune(W, H32, mode="nm", n=2, m=4, B=64)
    np.testing.assert_array_equal(Mg, orc.nm_mask(W, np.diag(H32), 2, 4))


@pytest.mark.parametrize("p", [0.5, 0.6])
@pytest.mark.parametrize("c,b,B", [(2563, 700, 256), (2560, 836, 512)])   # last blocks of 188 and 324 columns
def test_exact_ties_follow_row_major_order_for_many_rows(c, b, B, p):
    """As above where the mask of a block is chosen in a launch of its own (2560 rows and more)."""
    from tests.gpu_util import gpu_prune
    g = np.random.default_rng(2)
    W = g.choice(np.array([-2.0, -1.0, 0.5, 1.0, 2.0], dtype=np.float32), size=(c, b))
    H32 = np.diag(g.choice(np.array([1.0, 4.0], dtype=np.float32), size=b))
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=p, B=B, damp=0.01)
    assert info == 0
    Mref = orc.psi(W, np.diag(H32), orc.num_to_remove(p, c, b))
    np.testing.assert_array_equal(Mg, Mref)
    np.testing.assert_array_equal(Wg, W * (1 - Mref))


@pytest.mark.parametrize("need", [1, 5, 14])
def test_few_ties_at_the_threshold_in_later_blocks(need):
    """Distinct metrics except 15 equal ones exactly at the threshold, scattered over all blocks,
    of which `need` are removed: every block after the first resolves its threshold from the
    window the previous update counted and must rank the ties in (row, column) order over its
    residual.  Diagonal Hessian: no weight moves, so the mask is one global psi."""
    from tests.gpu_util import gpu_prune
    g = np.random.default_rng(3)
    c, b, N = 64, 512, 64 * 512
    vals = (np.arange(1, N + 1, dtype=np.float32) / np.float32(N))       # exact in fp32, distinct
    r = N // 2
    lo = r - need                                    # ranks lo+1 .. lo+15 become ties
    vals[lo:lo + 15] = vals[lo]
    W = (g.permutation(vals) * g.choice(np.array([-1.0, 1.0], dtype=np.float32), size=N)
         ).reshape(c, b).astype(np.float32)
    H32 = np.eye(b, dtype=np.float32)
    tie_cols = np.nonzero(np.abs(W) == vals[lo])[1]
    assert len(tie_cols) == 15 and len(set(tie_cols // 128)) >= 3      # ties in several blocks
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=0.5, B=128, damp=0.01)
    assert info == 0
    Mref = orc.psi(W, np.ones(b), r)
    assert int(Mref[np.abs(W) == vals[lo]].sum()) == need               # the cut is inside the ties
    np.testing.assert_array_equal(Mg, Mref)
    np.testing.assert_array_equal(Wg, W * (1 - Mref))


@pytest.mark.parametrize("mode", ["unstructured", "nm"])
def test_seventeen_row_tiles(mode):
    # 2176 rows = 17 row tiles of the trailing update: its tile order by XCD (bands of
    # ceil(17 / 8) = 3 row tiles, the last XCDs with a short band or none) is only used from 16
    # row tiles on.
    from tests.gpu_util import gpu_prune
    c, b = 2176, 384
    W, H32 = _layer(c, b, 1536, "f32", rho=0.7, seed=21)
    print(f"17 row tiles {mode}", flush=True)
    H = H32.astype(np.float64)
    if mode == "nm":
        Wg, Mg, info = gpu_prune(W, H32, mode="nm", n=2, m=4, B=128)
        Wo, Mo = orc.prune_nm(W, H, 2, 4, 128, 0.01)
        assert np.all(Mg.reshape(c, b // 4, 4).sum(axis=2) == 2)
    else:
        Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=0.5, B=128)
        Wo, Mo = orc.prune_unstructured(W, H, 0.5, 128, 0.01)
        assert int(Mg.sum()) == orc.num_to_remove(0.5, c, b)
    assert info == 0
    # fp32 against fp64 weights after the updates: a few near-ties may fall the other way
    assert np.mean(Mg != Mo) < 2e-4
    same = np.all(Mg == Mo, axis=1)
    assert same.mean() > 0.9
    assert _rel(Wg[same], Wo[same]) < 1e-3
    _check(W, H32, Wg, Mg, Wo, Mo, exact_mask=False)


def test_threshold_jumps_between_blocks():
    # Column blocks of very different scale: the global threshold moves by orders of magnitude
    # from block to block, far outside the window predicted from the previous block's, so every
    # block after the first takes the full radix passes; the third block loses all its 128
    # columns in every row (s = B), the second nearly none.
    from tests.gpu_util import gpu_prune
    W, H32 = _layer(96, 512, 2048, "f32", rho=0.0, seed=11)
    scale = np.repeat(np.array([1.0, 300.0, 0.01, 20.0], dtype=np.float32), 128)
    W = (W * scale).astype(np.float32)
    print("threshold jumps", flush=True)
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=0.5, B=128)
    assert info == 0
    Wo, Mo, margins = orc.prune_unstructured(W, H32.astype(np.float64), 0.5, 128, 0.01,
                                             return_margins=True)
    assert margins.min() > 2e-5, "seed has a near-tie; pick another"
    per_block = Mo.reshape(96, 4, 128).sum(axis=(0, 2))
    assert per_block[2] == 96 * 128 and per_block[1] < 96
    _check(W, H32, Wg, Mg, Wo, Mo)
    _, Mo64 = orc.prune_unstructured(W, H32.astype(np.float64), 0.5, 128, 0.01,
                                     metric_dtype=np.float64)
    np.testing.assert_array_equal(Mg, Mo64)


@pytest.mark.parametrize("growth", [1.002, 1.006, 1.02])
def test_threshold_drifts_steadily(growth):
    # Column blocks whose scale grows by a constant factor: the global threshold moves by a
    # steady step from block to block -- a fraction of the narrowest selection window, about its
    # half-width, and beyond the widest one -- so the sweep meets windows of every bin width and
    # blocks that fall back to the radix passes.
    from tests.gpu_util import gpu_prune
    from tests.fullsize_util import check_unstructured_rows
    c, b, B = 96, 2048, 128
    W, H32 = _layer(c, b, 4096, "f32", rho=0.0, seed=21)
    W = (W * (growth ** (np.arange(b) // B)).astype(np.float32)[None, :]).astype(np.float32)
    print(f"threshold drift, growth {growth} per block", flush=True)
    Wg, Mg, info, tau = gpu_prune(W, H32, mode="unstructured", p=0.5, B=B, tau=True)
    assert info == 0 and int(Mg.sum()) == c * b // 2
    H = H32.astype(np.float64)
    Wo, Mo = orc.prune_unstructured(W, H, 0.5, B, 0.01)
    step = np.abs(np.diff(tau)) / tau[:-1]
    print(f"  relative step of the threshold per block: median {np.median(step):.1e}, "
          f"max {step.max():.1e}; masks differ at {int((Mg != Mo).sum())} positions", flush=True)
    assert (Mg != Mo).mean() < 1e-4
    check_unstructured_rows(W, H, orc.inverse_factor(orc.damped(H, 0.01)), Wg.astype(np.float64), Mg,
                            tau, 0.5, B, 0.01, f"drift {growth}")


def test_sparsity_edge_values():
    from tests.gpu_util import gpu_prune
    W, H32 = _layer(16, 128, 512, "f32", seed=7)
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=0.0, B=64)
    assert Mg.sum() == 0
    np.testing.assert_array_equal(Wg, W)
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=0.6, B=64)
    assert int(Mg.sum()) == orc.num_to_remove(0.6, 16, 128)
    Wo, Mo = orc.prune_unstructured(W, H32.astype(np.float64), 0.6, 64, 0.01)
    np.testing.assert_array_equal(Mg, Mo)


# --------------------------------------------------------------------------- dtypes, determinism
def test_fp16_weights_cast_output_and_determinism():
    from tests.gpu_util import gpu_prune
    W, H32 = _layer(128, 512, 2048, "f16", seed=8)
    Wg, Mg, info, Wc = gpu_prune(W, H32, mode="nm", n=2, m=4, B=128, cast=True)
    assert Wc.dtype == np.float16
    np.testing.assert_array_equal(Wc, Wg.astype(np.float16))
    Wo, Mo = orc.prune_nm(W, H32.astype(np.float64), 2, 4, 128, 0.01)
    ok = np.all(Mg == Mo, axis=1)
    assert ok.mean() > 0.98
    assert _rel(Wg[ok], Wo[ok]) < 1e-3
    W2, M2, _, _ = gpu_prune(W, H32, mode="nm", n=2, m=4, B=128, cast=True)
    np.testing.assert_array_equal(W2, Wg)
    np.testing.assert_array_equal(M2, Mg)
    a = gpu_prune(W, H32, mode="unstructured", p=0.5, B=128)
    b_ = gpu_prune(W, H32, mode="unstructured", p=0.5, B=128)
    np.testing.assert_array_equal(a[0], b_[0])
    np.testing.assert_array_equal(a[1], b_[1])


# --------------------------------------------------------------------------- several tiles
@pytest.mark.parametrize("mode", ["unstructured", "nm"])
def test_medium_layer_teacher_forced(mode):
    # 300 x 1024 spans several 128-tiles in both directions and 8 blocks.  The free-running
    # mask may differ from the float64 oracle at near-ties only; W_hat is compared under the
    # GPU's own mask (the oracle re-run with that mask forced).
    from tests.gpu_util import gpu_prune
    c, b, B = 300, 1024, 128
    W, H32 = _layer(c, b, 4096, "f16", seed=9)
    H = H32.astype(np.float64)
    print(f"medium {mode}", flush=True)
    if mode == "unstructured":
        Wg, Mg, info = gpu_prune(W, H32, mode=mode, p=0.5, B=B)
        Wo, Mo = orc.prune_fast(W, H, mode=mode, p=0.5, B=B, damp=0.01)
        assert int(Mg.sum()) == c * b // 2
    else:
        Wg, Mg, info = gpu_prune(W, H32, mode=mode, n=2, m=4, B=B)
        Wo, Mo = orc.prune_fast(W, H, mode=mode, n=2, m=4, B=B, damp=0.01)
        assert np.all(Mg.reshape(c, b // 4, 4).sum(axis=2) == 2)
    assert info == 0
    assert (Mg != Mo).mean() < 1e-4
    Wt, _ = orc.prune_fast(W, H, mode=mode, p=0.5, n=2, m=4, B=B, damp=0.01, mask_in=Mg)
    assert _rel(Wg, Wt) < 1e-3
    eo = orc.reconstruction_error(W, Wo, H)
    eg = orc.reconstruction_error(W, Wg.astype(np.float64), H)
    assert abs(eg - eo) <= 0.01 * eo


@pytest.mark.parametrize("B", [64, 128, 256])
def test_singular_row_system_is_reported(B):
    # A factor with a zero column makes G = U_kk^T U_kk singular in that column: the one row
    # whose mask contains it must be reported as -(row + 1); the three block sizes reach the
    # three per-row solvers (register tiles, 128 threads, LDS tiles).
    from tests.gpu_util import gpu_prune, gpu_factor
    c, b, bad_row, bad_col = 12, 2 * B, 3, 5
    W, H32 = _layer(c, b, 4 * b, "f32", seed=B)
    U, xn2, info = gpu_factor(H32, 0.01)
    assert info == 0
    U[:, bad_col] = 0.0
    rng = np.random.default_rng(B)
    M = (rng.random((c, b)) < 0.6).astype(np.uint8)
    M[:, bad_col] = 0
    M[bad_row, bad_col] = 1
    print(f"singular system B={B}", flush=True)
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=0.5, B=B, mask_in=M, U=U, xnorm2=xn2)
    assert info == -(bad_row + 1)
    np.testing.assert_array_equal(Mg, M)
    ok = np.arange(c) != bad_row
    assert np.all(np.isfinite(Wg[ok]))
    assert np.all(Wg[ok][M[ok] == 1] == 0.0)


@pytest.mark.parametrize("p", [0.72, 0.85])
def test_block128_rows_split_between_two_solvers(p):
    # B = 128 unstructured: rows with at most 96 removed weights in a block go to the
    # one-wavefront matrix-core solver, the others to the 128-thread one.  p = 0.72 puts rows on
    # both sides of that limit in every block, p = 0.85 nearly all of them above it.
    from tests.gpu_util import gpu_prune
    c, b = 192, 512
    W, H32 = _layer(c, b, 2048, "f32", rho=0.7, seed=77)
    print(f"split solvers p={p}", flush=True)
    Wg, Mg, info = gpu_prune(W, H32, mode="unstructured", p=p, B=128)
    assert info == 0
    assert int(Mg.sum()) == orc.num_to_remove(p, c, b)
    per_block = Mg.reshape(c, b // 128, 128).sum(axis=2)
    assert per_block.max() > 96
    if p < 0.8:
        assert per_block.min() <= 96
    H = H32.astype(np.float64)
    Wt, _ = orc.prune_fast(W, H, mode="unstructured", p=p, B=128, damp=0.01, mask_in=Mg)
    assert np.all(Wg[Mg == 1] == 0.0)
    assert _rel(Wg, Wt) < 1e-3
    _, Mo = orc.prune_fast(W, H, mode="unstructured", p=p, B=128, damp=0.01)
    assert (Mg != Mo).mean() < 1e-3


# --------------------------------------------------------------------------- conditioning
@pytest.mark.parametrize("T,rho,damp,mode,B", [
    (512, 0.7, 0.01, "nm", 128),              # fewer tokens than channels: H is rank deficient
    (256, 0.9, 0.01, "unstructured", 128),    # rank 256 of 1024, strongly correlated channels
    (4096, 0.95, 0.001, "unstructured", 256),  # small damping, condition number > 1e4
    (4096, 0.7, 0.0001, "nm", 128),
])
def test_ill_conditioned_hessians(T, rho, damp, mode, B):
    """Damping is all that keeps these Hessians positive definite (condition numbers of the
    damped matrix 5e3 .. 4e4); the fp32 factor and solves must still give the oracle's W_hat."""
    from tests.gpu_util import gpu_prune
    c, b = 256, 1024
    W, H32 = _layer(c, b, T, "f16", rho=rho, seed=5)
    H = H32.astype(np.float64)
    kw = dict(n=2, m=4) if mode == "nm" else dict(p=0.5)
    print(f"ill-conditioned {mode} T={T} rho={rho} damping={damp} B={B}", flush=True)
    Wg, Mg, info = gpu_prune(W, H32, mode=mode, B=B, damp=damp, **kw)
    assert info == 0
    Wt, _ = orc.prune_fast(W, H, mode=mode, B=B, damp=damp, mask_in=Mg, **kw)
    assert np.all(Wg[Mg == 1] == 0.0)
    assert _rel(Wg, Wt) < 1e-3
    eo = orc.reconstruction_error(W, Wt, H)
    eg = orc.reconstruction_error(W, Wg.astype(np.float64), H)
    assert abs(eg - eo) <= 0.01 * eo


@pytest.mark.parametrize("mode", ["unstructured", "nm"])
def test_dead_input_channels(mode):
    """Input channels that are zero in every calibration token: H_jj = 0, so the metric of their
    weights is 0 and they go first (ties in (row, column) order); the damping alone keeps the
    Hessian positive definite.  No special case anywhere: masks as the oracle's, W_hat within
    the usual bound."""
    from tests.gpu_util import gpu_prune
    c, b, T, B = 96, 512, 2048, 128
    spec = LayerSpec("t", c=c, b=b, tokens=T, dtype="f16", rho=0.7, k_mix=16, seed=12)
    W, X = make_weight(spec), make_calibration(spec)
    dead = np.array([0, 5, 6, 130, 255, 256, 300, 511])        # 5 and 6 share a group of four
    X[:, dead] = 0
    H32 = orc.hessian(X).astype(np.float32)
    H = H32.astype(np.float64)
    assert np.all(np.diag(H)[dead] == 0.0)
    kw = dict(n=2, m=4) if mode == "nm" else dict(p=0.5)
    Wg, Mg, info = gpu_prune(W, H32, mode=mode, B=B, **kw)
    assert info == 0
    assert Mg[:, dead].all()                                   # every weight of a dead channel goes
    if mode == "nm":
        assert np.all(Mg.reshape(c, b // 4, 4).sum(axis=2) == 2)
        assert not Mg[:, [4, 7]].any()                         # the group 4..7 is used up by 5 and 6
    else:
        assert int(Mg.sum()) == c * b // 2
    Wo, Mo = orc.prune_fast(W, H, mode=mode, B=B, damp=0.01, **kw)
    ndiff = int((Mg != Mo).sum())
    assert ndiff <= 4, ndiff                                   # near-ties only (none at the dead channels)
    np.testing.assert_array_equal(Mg[:, dead], Mo[:, dead])
    Wt, _ = orc.prune_fast(W, H, mode=mode, B=B, damp=0.01, mask_in=Mg, **kw)
    assert np.all(Wg[Mg == 1] == 0.0)
    assert _rel(Wg, Wt) < 1e-3


# --------------------------------------------------------------------------- invariances
@pytest.mark.parametrize("mode", ["unstructured", "nm"])
def test_hessian_scale_does_not_matter(mode):
    """The update u R_hat^{-1} R and the order of the metric are unchanged by H -> kappa H when
    the damping is relative (Sec. 4.1 / 4.2: H enters as 2 X X^T, (2/d) sum or X X^T alike).
    With kappa a power of four every intermediate scales exactly (the factor by the power of
    two sqrt(kappa)), so the results are identical bit for bit."""
    from tests.gpu_util import gpu_prune
    W, H32 = _layer(200, 640, 2560, "f16", rho=0.7, seed=21)
    kw = dict(n=2, m=4) if mode == "nm" else dict(p=0.5)
    W1, M1, i1 = gpu_prune(W, H32, mode=mode, B=128, **kw)
    W2, M2, i2 = gpu_prune(W, (4.0 * H32).astype(np.float32), mode=mode, B=128, **kw)
    W3, M3, i3 = gpu_prune(W, (0.0625 * H32).astype(np.float32), mode=mode, B=128, **kw)
    assert i1 == i2 == i3 == 0
    np.testing.assert_array_equal(M1, M2)
    np.testing.assert_array_equal(W1, W2)
    np.testing.assert_array_equal(M1, M3)
    np.testing.assert_array_equal(W1, W3)


@pytest.mark.parametrize("kappa", [2.0 ** 80, 2.0 ** -80])
@pytest.mark.parametrize("mode,B,kw", [
    ("nm", 128, dict(n=2, m=4)), ("unstructured", 128, dict(p=0.5)),    # one wavefront per row
    ("nm", 256, dict(n=2, m=4)), ("unstructured", 256, dict(p=0.6)),    # tiles, complement form
    ("structured", 128, dict(p=0.3, alpha=0.1))])
def test_hessian_of_any_scale(mode, B, kw, kappa):
    """As above, at scales where the product of two pivots leaves the range of fp32."""
    from tests.gpu_util import gpu_prune
    W, H32 = _layer(200, 640, 2560, "f16", rho=0.7, seed=21)
    W1, M1, i1 = gpu_prune(W, H32, mode=mode, B=B, **kw)
    W2, M2, i2 = gpu_prune(W, (kappa * H32).astype(np.float32), mode=mode, B=B, **kw)
    assert i1 == i2 == 0
    np.testing.assert_array_equal(M1, M2)
    np.testing.assert_array_equal(W1, W2)


def test_nm_rows_are_independent():
    """n:m: rows only meet in the shared inverse, so permuting the rows of W permutes the rows
    of (W_hat, M) and changes nothing else (bit for bit: a row's arithmetic does not depend on
    which tile or wavefront it lands in)."""
    from tests.gpu_util import gpu_prune
    W, H32 = _layer(300, 512, 2048, "f16", rho=0.7, seed=22)
    perm = np.random.default_rng(0).permutation(W.shape[0])
    W1, M1, _ = gpu_prune(W, H32, mode="nm", n=2, m=4, B=128)
    W2, M2, _ = gpu_prune(np.ascontiguousarray(W[perm]), H32, mode="nm", n=2, m=4, B=128)
    np.testing.assert_array_equal(M1[perm], M2)
    np.testing.assert_array_equal(W1[perm], W2)


@pytest.mark.parametrize("mode,kw,c,b,B", [
    ("nm", dict(n=2, m=4), 130, 1160, 128),            # two super-blocks, the second with one short block
    ("nm", dict(n=4, m=8), 37, 2600, 8),               # many super-blocks of a few columns
    ("nm", dict(n=2, m=4), 40, 780, 256),              # tiled solver, four tile rows
    ("nm", dict(n=4, m=8), 21, 1064, 512),             # eight, then one of four unknowns
    ("unstructured", dict(p=0.5), 130, 520, 128),
    ("unstructured", dict(p=0.7), 33, 650, 256),       # complement form, tiled solver
    ("unstructured", dict(p=0.6), 2561, 512, 256),     # complement form for many rows
    ("unstructured", dict(p=0.5), 65, 333, 100)])      # unaligned rows
def test_scales_of_channels_and_rows(mode, kw, c, b, B):
    """The sweep's products see scaled columns and rows.  Undamped, H -> D H D, W -> R W D^-1 with
    powers of two changes no metric's order within a row (n:m) or at all (R = 1), and every value of the
    result by exactly that factor: masks equal, weights equal bit for bit."""
    from tests.gpu_util import gpu_prune
    W, H32 = _layer(c, b, 2 * b, "f32", seed=b + c)
    g = np.random.default_rng(c)
    d = np.ldexp(np.float32(1.0), g.integers(-20, 21, size=b))
    r = np.ldexp(np.float32(1.0), g.integers(-20, 21, size=c) if mode == "nm" else np.zeros(c, int))
    W1, M1, i1 = gpu_prune(W, H32, mode=mode, B=B, damp=0.0, **kw)
    W2, M2, i2 = gpu_prune((r[:, None] * W / d[None, :]).astype(np.float32),
                           (H32 * d[:, None] * d[None, :]).astype(np.float32), mode=mode, B=B, damp=0.0, **kw)
    assert i1 == i2 == 0
    np.testing.assert_array_equal(M1, M2)
    np.testing.assert_array_equal(W1, W2 / r[:, None] * d[None, :])


def test_given_factor_of_any_scale():
    """A factor of the caller whose columns differ by 2^+-40 (scales come from the factor itself)."""
    from tests.gpu_util import gpu_prune, gpu_factor
    c, b, B = 70, 400, 64
    W, H32 = _layer(c, b, 4 * b, "f32", seed=11)
    U, xn2, info = gpu_factor(H32, 0.0)
    assert info == 0
    d = np.ldexp(np.float32(1.0), np.random.default_rng(3).integers(-40, 41, size=b))
    W1, M1, i1 = gpu_prune(W, H32, mode="nm", n=2, m=4, B=B, U=U, xnorm2=xn2)
    W2, M2, i2 = gpu_prune((W / d[None, :]).astype(np.float32), H32, mode="nm", n=2, m=4, B=B, U=U / d[None, :],
                           xnorm2=xn2 * d * d)
    assert i1 == i2 == 0
    np.testing.assert_array_equal(M1, M2)
    np.testing.assert_array_equal(W1, W2 * d[None, :])


@pytest.mark.parametrize("c,b,B", [(130, 256, 128), (70, 330, 110), (129, 390, 64)])
@pytest.mark.parametrize("mode", ["nm", "unstructured"])
def test_results_anywhere_in_memory(mode, c, b, B):
    """W_out and mask_out at element-aligned addresses, rows of any length: pairs of values and 16-byte
    pieces are fetched unaligned.  Equal bits to a call with aligned buffers, nothing written around."""
    import torch
    import paper_2504_05346_amd as th
    W, H32 = _layer(c, b, 2 * b, "f32", seed=b)
    o = th.PruneOpts(mode=th.THANOS_NM if mode == "nm" else th.THANOS_UNSTRUCTURED, sparsity=0.5, n=1, m=2,
                     block_size=B, damping=0.01, outlier_fraction=0.1 if mode == "nm" else 0.0)
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H32).cuda()
    ws = torch.empty((th.thanos_prune_workspace_bytes(c, b, o),), dtype=torch.uint8, device="cuda")
    info = torch.zeros((1,), dtype=torch.int32, device="cuda")
    got = []
    for off in (0, 1, 3):
        buf = torch.full((c * b + 8,), 7.5, device="cuda")
        mb = torch.full((c * b + 8,), 9, dtype=torch.uint8, device="cuda")
        out, mask = buf[off:off + c * b].view(c, b), mb[off:off + c * b].view(c, b)
        th.thanos_prune_layer(Wd, Hd, o, out, None, mask, ws, info)
        torch.cuda.synchronize()
        assert int(info.item()) == 0
        got.append((out.cpu().numpy(), mask.cpu().numpy()))
        for t, v in ((buf, 7.5), (mb, 9)):
            assert bool((t[:off] == v).all()) and bool((t[off + c * b:] == v).all())
    for w, m in got[1:]:
        np.testing.assert_array_equal(w, got[0][0])
        np.testing.assert_array_equal(m, got[0][1])


@pytest.mark.parametrize("route,c,b,B", [
    ("mask", 96, 1300, 128),           # reductions of 1024 right of the super-block
    ("mask", 130, 2301, 256),          # of 2048, two row tiles per block, odd rows
    ("mask", 40, 900, 96), ("mask", 33, 533, 24),
    ("mask", 50, 1001, 110),           # reductions of 110 and 880: no whole slabs, multipliers of odd alignment
    ("unstructured", 129, 900, 128), ("unstructured", 70, 777, 200), ("unstructured", 70, 1201, 512),
    ("unstructured", 50, 601, 75)])
def test_update_of_weakly_coupled_columns(route, c, b, B):
    """A wide, nearly diagonal H: couplings of 2^-18 between the columns, 2^-8 in every sixteenth.  The weights
    right of the removed ones start at (next to) nothing, so that their results are the update's product
    alone.  Each column is as exact as fp32: block row, solve and product round at 2^-24 each, sums of up to
    2048 values of either sign gain less than 8 times that (measured 3 to 8e-7); with a scale of P taken from a
    bound instead of its values the weak columns were off by 2e-5 to 7e-4."""
    from tests.gpu_util import gpu_prune
    g = np.random.default_rng(b)
    U = np.triu(2.0 ** -18 * g.standard_normal((b, b)), 1)
    U[:, 5::16] *= 2.0 ** 10
    U = (np.triu(U, 1) + np.diag(1.0 + g.random(b))).astype(np.float32)
    first = B if route == "unstructured" else 8 * B
    W = np.full((c, b), 1e-30, dtype=np.float32)
    W[:, :first] = g.standard_normal((c, first))
    if route == "mask":
        M = np.zeros((c, b), dtype=np.uint8)
        M[:, :first] = g.random((c, first)) < 0.5
        Wg, Mg, info = gpu_prune(W, None, mode="unstructured", p=0.5, B=B, mask_in=M, U=U, xnorm2=np.ones(b))
    else:  # channel norms that keep the selection in the first block
        xn2 = np.where(np.arange(b) < first, 1e-30, 1e36)
        Wg, Mg, info = gpu_prune(W, None, mode="unstructured", p=round(0.5 * B / b, 4), B=B, U=U, xnorm2=xn2)
        assert Mg[:, :first].any(axis=1).all() and not Mg[:, first:].any()
    assert info == 0
    Wt, _ = orc.prune_fast(W, np.eye(b), mode="unstructured", p=0.0, B=B, damp=0.0, mask_in=Mg,
                           U=U.astype(np.float64))
    e = np.linalg.norm((Wg - Wt)[:, first:], axis=0) / np.linalg.norm(Wt[:, first:], axis=0)
    print(f"{route} {c}x{b} B={B}: worst column {e.max():.2e}", flush=True)
    assert e.max() <= 2.0 ** -20


def _near_identity(b, seed, spread=0.25):
    """H = D (I + E) D: eigenvalues of I + E within 1 +- 2 spread, channel scales log-normal.  float32, symmetric."""
    g = np.random.default_rng(seed)
    E = np.triu(g.standard_normal((b, b)) * (spread / np.sqrt(b)), 1)
    d = np.exp(g.standard_normal(b))
    return ((np.eye(b) + E + E.T) * d[:, None] * d[None, :]).astype(np.float32)


@pytest.mark.parametrize("mode,kw,B", [
    ("nm", dict(n=2, m=4), 64), ("nm", dict(n=2, m=4), 128),
    ("nm", dict(n=2, m=4), 256), ("nm", dict(n=2, m=4), 512),    # tiled solver: 128 and 256 unknowns
    ("unstructured", dict(p=0.5), 128), ("unstructured", dict(p=0.4), 256),
    ("unstructured", dict(p=0.7), 256)])                          # through the complement
def test_single_block_is_as_exact_as_fp32(mode, kw, B):
    """One block, well-conditioned: what the call adds to the kept weights, relative to float64 under the same
    mask.  Factor, block rows, solve and update round at 2^-24 each, in sums of up to B values of either sign
    (3e-7 for the factor, about the same for the rest; measured 5 to 8e-7)."""
    from tests.gpu_util import gpu_prune
    H32 = _near_identity(B, seed=B)
    W = np.random.default_rng(7).standard_normal((200, B)).astype(np.float32)
    W /= np.sqrt(np.diag(H32))
    Wg, Mg, info = gpu_prune(W, H32, mode=mode, B=B, damp=0.0, **kw)
    assert info == 0
    Wt, _ = orc.prune_fast(W, H32.astype(np.float64), mode="unstructured", p=0.0, B=B, damp=0.0, mask_in=Mg)
    kept = Mg == 0
    d = np.sqrt(np.diag(H32).astype(np.float64))[None, :]
    e = np.linalg.norm(((Wg - Wt) * d)[kept]) / np.linalg.norm(((Wt - W) * d)[kept])
    print(f"{mode} B={B}: {e:.2e}", flush=True)
    assert e <= 2.0 ** -20


def test_factor_beside_the_row_losses_has_the_same_bits():
    """With outlier rows the factorisation's products take one LDS buffer instead of two (the row losses run
    beside them): the result is that of the factor computed alone and passed in, bit for bit."""
    from tests.gpu_util import gpu_prune, gpu_factor
    b, c = 3200, 96
    H32 = _near_identity(b, seed=5)
    W = np.random.default_rng(8).standard_normal((c, b)).astype(np.float32)
    U, xn2, info = gpu_factor(H32, 0.01)
    assert info == 0
    W1, M1, i1 = gpu_prune(W, H32, mode="nm", n=4, m=8, B=128, alpha=0.1)
    W2, M2, i2 = gpu_prune(W, H32, mode="nm", n=4, m=8, B=128, alpha=0.1, U=U, xnorm2=xn2)
    assert i1 == i2 == 0 and (M1.sum(axis=1) == 0).sum() == 10
    np.testing.assert_array_equal(M1, M2)
    np.testing.assert_array_equal(W1, W2)


@pytest.mark.parametrize("mode,kw,c,b,B", [
    ("nm", dict(n=2, m=4), 31, 129 * 4, 128),          # fewer rows than a tile, 516 columns: 4 in the last strip
    ("nm", dict(n=2, m=4), 33, 640, 16),               # right of the super-block: eight exponents per column of P
    ("nm", dict(n=2, m=4), 65, 1300, 128),             # a super-block and a bit
    ("nm", dict(n=4, m=8), 64, 1024, 512),             # reductions of 512
    ("unstructured", dict(p=0.5), 1, 384, 128),
    ("unstructured", dict(p=0.5), 97, 515, 128),       # rows of any alignment, ragged last block
    ("unstructured", dict(p=0.4), 130, 768, 256),
    ("unstructured", dict(p=0.5), 1024, 1029, 128),    # 32 x 9 strips in the first block
    ("nm", dict(n=2, m=4), 1056, 1024, 128),           # 33 x 8 strips, then 33 x 7: both kernels
    ("unstructured", dict(p=0.5), 1921, 640, 128)])    # 61 x 5, then 61 x 4, with 16 tile rows: both kernels
def test_update_of_few_tiles(mode, kw, c, b, B):
    """What the sweep adds to the kept weights, relative to float64 under the same mask, where the updates are
    launches of few tiles: well-conditioned H, so that factor, block rows, solve and update are off by some 2^-24
    each, in sums of up to b values of either sign; 2^-20 as for single blocks, times two for the blocks in turn."""
    from tests.gpu_util import gpu_prune
    H32 = _near_identity(b, seed=b + B)
    W = np.random.default_rng(c).standard_normal((c, b)).astype(np.float32)
    W /= np.sqrt(np.diag(H32))
    print(f"few tiles {mode} {c}x{b} B={B}", flush=True)
    Wg, Mg, info = gpu_prune(W, H32, mode=mode, B=B, damp=0.0, **kw)
    assert info == 0
    if mode == "unstructured":
        assert int(Mg.sum()) == orc.num_to_remove(kw["p"], c, b)
    Wt, _ = orc.prune_fast(W, H32.astype(np.float64), mode="unstructured", p=0.0, B=B, damp=0.0, mask_in=Mg)
    kept = Mg == 0
    d = np.sqrt(np.diag(H32).astype(np.float64))[None, :]
    e = np.linalg.norm(((Wg - Wt) * d)[kept]) / np.linalg.norm(((Wt - W) * d)[kept])
    print(f"  {e:.2e}", flush=True)
    assert np.all(Wg[Mg == 1] == 0.0) and e <= 2.0 ** -19


@pytest.mark.parametrize("c,b,s", [
    (130, 200, 1), (33, 200, 64), (130, 200, 65),     # reductions up to 64: three-way split; then two-way
    (64, 300, 290), (1, 257, 256),                    # no room for whole slabs of 32 in the buffer of the removed columns
    (131, 1029, 400), (257, 1300, 1000)])             # more columns than the short routes of the gathers take
def test_structured_update_is_as_exact_as_fp32(c, b, s):
    """What the update adds to the kept columns, relative to float64 with the same columns removed, on a
    well-conditioned H: factor and two products of up to 1000 values round at 2^-24 each, sums of either sign gain
    less than 16 times that; and the kept weights themselves are rounded once more, at 2^-24 of their own size (with
    one column removed they are 60 times as large as what is added)."""
    from tests.gpu_util import gpu_prune
    H32 = _near_identity(b, seed=b + s)
    W = np.random.default_rng(c).standard_normal((c, b)).astype(np.float32)
    W /= np.sqrt(np.diag(H32))
    print(f"structured {c}x{b} s={s}", flush=True)
    Wg, Mg, info = gpu_prune(W, H32, mode="structured", p=(s - 0.5) / b, damp=0.0)
    assert info == 0 and (Mg == Mg[0]).all() and Mg[0].sum() == s
    Q, K = Mg[0] == 1, Mg[0] == 0
    Hi = np.linalg.inv(H32.astype(np.float64))
    D = -np.linalg.solve(Hi[np.ix_(Q, Q)].T, W[:, Q].astype(np.float64).T).T @ Hi[np.ix_(Q, K)]
    d = np.sqrt(np.diag(H32).astype(np.float64))[K]
    e = np.linalg.norm((Wg[:, K] - (W[:, K] + D)) * d) / np.linalg.norm(D * d)
    print(f"  {e:.2e}", flush=True)
    assert np.all(Wg[:, Q] == 0.0)
    assert e <= 2.0 ** -20 + 2.0 ** -24 * np.linalg.norm(W[:, K] * d) / np.linalg.norm(D * d)


@pytest.mark.parametrize("mode,kw,c,b", [
    ("nm", dict(n=2, m=4, B=128), 130, 516), ("nm", dict(n=2, m=4, B=128), 40, 1300),
    ("structured", dict(p=0.3), 130, 515), ("structured", dict(p=0.4), 70, 1101)])
def test_row_losses_of_channels_of_any_scale(mode, kw, c, b):
    """Outlier rows, undamped: H -> D H D, W -> W D^-1 with powers of two over 2^+-20 leaves every loss as it is, so the
    same rows stay, and every weight changes by its factor, bit for bit."""
    from tests.gpu_util import gpu_prune
    W, H32 = _layer(c, b, 2 * b, "f32", seed=b)
    d = np.ldexp(np.float32(1.0), np.random.default_rng(c).integers(-20, 21, size=b))
    print(f"row losses {mode} {c}x{b}", flush=True)
    W1, M1, i1 = gpu_prune(W, H32, mode=mode, alpha=0.25, damp=0.0, **kw)
    W2, M2, i2 = gpu_prune((W / d[None, :]).astype(np.float32), (H32 * d[:, None] * d[None, :]).astype(np.float32),
                           mode=mode, alpha=0.25, damp=0.0, **kw)
    assert i1 == i2 == 0
    h = orc.row_losses(W.astype(np.float64), H32.astype(np.float64))
    stay = ~M1.any(axis=1)
    assert stay.sum() == orc.num_outlier_rows(0.25, c) and h[stay].min() > h[~stay].max() * (1 - 1e-6)
    np.testing.assert_array_equal(M1, M2)
    np.testing.assert_array_equal(W1, W2 * d[None, :])


def _same_rows_stay(W, H32, M, alpha):
    """The rows that were left alone are those with the largest losses in float64 (ties to 1e-6)."""
    h = orc.row_losses(W.astype(np.float64), H32.astype(np.float64))
    stay = ~M.any(axis=1)
    assert stay.sum() == orc.num_outlier_rows(alpha, W.shape[0])
    assert h[stay].min() > h[~stay].max() - 1e-6 * np.abs(h).max()


@pytest.mark.parametrize("mode,kw,c,b,given", [
    ("nm", dict(n=2, m=4, B=128), 130, 516, False), ("nm", dict(n=2, m=4, B=128), 40, 1300, False),
    ("nm", dict(n=2, m=4, B=128), 130, 516, True), ("nm", dict(n=2, m=4, B=128), 40, 1300, True),
    ("structured", dict(p=0.3), 130, 515, False), ("structured", dict(p=0.4), 70, 1101, False)])
def test_row_losses_beside_channels_without_activations(mode, kw, c, b, given):
    """Zero rows and columns of H under large weights, the others' values 2^-60 times as large as they were: what a
    channel without activations weighs has no part in a loss, and none in its rounding."""
    from tests.gpu_util import gpu_factor, gpu_prune
    W, H32 = _layer(c, b, 2 * b, "f32", seed=b)
    g = np.random.default_rng(c)
    dead = g.permutation(b)[:b // 50]
    W[:, dead] = 50 * g.standard_normal((c, dead.size))
    H32[dead] = H32[:, dead] = 0.0
    H32 *= np.float32(2.0 ** -60)
    how = dict(kw)
    if given:
        U, xn2, info = gpu_factor(H32, 0.01)
        assert info == 0
        how.update(U=U, xnorm2=xn2)
    print(f"no activations {mode} {c}x{b} given={given}", flush=True)
    _, M, info = gpu_prune(W, H32, mode=mode, alpha=0.25, damp=0.01, **how)
    assert info == 0
    _same_rows_stay(W, H32, M, 0.25)


@pytest.mark.parametrize("mode,kw,c,b,given", [
    ("nm", dict(n=2, m=4, B=128), 130, 516, False), ("nm", dict(n=2, m=4, B=128), 41, 1300, True),
    ("structured", dict(p=0.3), 131, 515, False), ("structured", dict(p=0.4), 70, 1101, False)])
@pytest.mark.parametrize("zeros", [False, True])
def test_row_losses_of_an_indefinite_hessian(mode, kw, c, b, given, zeros):
    """Elements of H that are far larger than their channels' diagonal, some of it zero and one negative: positive
    definite only with its damping.  The losses are what H gives, of either sign.  zeros: an element between two
    channels of zero diagonal, which no scale of theirs brings into the range of fp32."""
    from tests.gpu_util import gpu_factor, gpu_prune
    W, H32 = _layer(c, b, 2 * b, "f32", seed=b)
    g = np.random.default_rng(c)
    at = g.permutation(b)[:8].reshape(4, 2)
    top = float(np.diag(H32).max())
    for k, (i, j) in enumerate(at):
        H32[i, j] = H32[j, i] = (-1) ** k * 300.0 * top
    if zeros:
        H32[at[2, 0], at[2, 0]] = H32[at[2, 1], at[2, 1]] = 0.0
    H32[at[0, 0], at[0, 0]] = 0.0
    H32[at[1, 1], at[1, 1]] *= -1.0
    damp = 2000.0 * top / float(np.diag(H32).mean())
    how = dict(kw)
    if given:
        U, xn2, info = gpu_factor(H32, damp)
        assert info == 0
        how.update(U=U, xnorm2=xn2)
    print(f"indefinite {mode} {c}x{b} given={given}", flush=True)
    _, M, info = gpu_prune(W, H32, mode=mode, alpha=0.25, damp=damp, **how)
    assert info == 0
    _same_rows_stay(W, H32, M, 0.25)


@pytest.mark.parametrize("e", [15, 20, 24])
def test_structured_update_of_groups_of_different_size(e):
    """Two groups of channels that do not correlate, and rows whose weights in one of them are 2^e times smaller:
    what these gain is as exact as in test_structured_update_is_as_exact_as_fp32."""
    from tests.gpu_util import gpu_prune
    c, b, s = 64, 512, 205
    g = np.random.default_rng(5)
    H32 = _near_identity(b, seed=3)
    first = np.zeros(b, dtype=bool)
    first[g.permutation(b)[:b // 2]] = True
    H32[np.ix_(first, ~first)] = H32[np.ix_(~first, first)] = 0
    W = (g.standard_normal((c, b)) / np.sqrt(np.diag(H32))).astype(np.float32)
    even = np.arange(c) % 2 == 0
    W[np.ix_(even, ~first)] *= np.float32(2.0 ** -e)
    W[np.ix_(~even, first)] *= np.float32(2.0 ** -e)
    print(f"groups 2^{e} apart", flush=True)
    Wg, Mg, info = gpu_prune(W, H32, mode="structured", p=(s - 0.5) / b, damp=0.0)
    assert info == 0 and (Mg == Mg[0]).all() and Mg[0].sum() == s
    Q, K = Mg[0] == 1, Mg[0] == 0
    assert (Q & first).sum() > 64 and (Q & ~first).sum() > 64
    Hi = np.linalg.inv(H32.astype(np.float64))
    D = -np.linalg.solve(Hi[np.ix_(Q, Q)].T, W[:, Q].astype(np.float64).T).T @ Hi[np.ix_(Q, K)]
    d = np.sqrt(np.diag(H32).astype(np.float64))[K]
    for rows, chans in ((even, ~first[K]), (~even, first[K])):  # the small weights
        at = np.ix_(rows, chans)
        err = np.linalg.norm(((Wg[:, K] - (W[:, K] + D)) * d)[at])
        added, kept = np.linalg.norm((D * d)[at]), np.linalg.norm((W[:, K] * d)[at])
        print(f"  {err / added:.2e}", flush=True)
        assert err / added <= 2.0 ** -20 + 2.0 ** -24 * kept / added


def test_structured_and_row_losses_beyond_32768_columns():
    """Rows that do not fit the LDS: permuted and gathered from memory.  H = E + v v^T with E diagonal, for which
    everything has a closed form: the losses of columns and rows, and the update W_Q H_QK H_KK^-1 of the kept columns,
    which is v_Q v_K^T E_K^-1 / (1 + v_K^T E_K^-1 v_K).  Weights along E^-1 v, so that the update is about as large
    as they are; its sums over 10^4 values of one sign, 600 partial sums of 16, round by up to sqrt(600 / 3) 2^-24 in
    each of the two products and about as much in the factor: 2^-19 instead of the 2^-20 of sums of either sign."""
    import torch
    import paper_2504_05346_amd as th
    c, b, p, alpha = 40, 33001, 0.3, 0.1
    gen = torch.Generator(device="cuda").manual_seed(33)
    E = torch.exp(torch.randn(b, generator=gen, device="cuda"))
    v = torch.randn(b, generator=gen, device="cuda").sign() * E.sqrt() * (2.0 / b ** 0.5)  # v^T E^-1 v = 4
    H = torch.diag(E).addr_(v, v)
    E = H.diagonal().double() - v.double() ** 2  # what the rounded diagonal stands for
    W = torch.randn((c, b), generator=gen, device="cuda") * (0.5 / E.float().sqrt())
    W += torch.randn((c, 1), generator=gen, device="cuda") * (v / E.float()) * b ** 0.5 / 2
    o = th.PruneOpts(mode=th.THANOS_STRUCTURED, sparsity=p, damping=0.0, outlier_fraction=alpha, block_size=128)
    ws = torch.empty((th.thanos_prune_workspace_bytes(c, b, o),), dtype=torch.uint8, device="cuda")
    Wo, M = torch.empty((c, b), device="cuda"), torch.empty((c, b), dtype=torch.uint8, device="cuda")
    info = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    print(f"structured {c}x{b}", flush=True)
    th.thanos_prune_layer(W, H, o, Wo, None, M, ws, info)
    torch.cuda.synchronize()
    assert int(info) == 0
    W, Wo, E, v = (t.double().cpu().numpy() for t in (W, Wo, E, v))
    M = M.cpu().numpy().astype(bool)
    h = (W * W) @ E + (W @ v) ** 2
    rows = M.any(axis=1)
    assert (~rows).sum() == orc.num_outlier_rows(alpha, c) and h[~rows].min() > h[rows].max() * (1 - 1e-6)
    Q, K = M[rows][0], ~M[rows][0]
    assert (M[rows] == Q).all()
    col = (E + v * v) * (W[rows] ** 2).sum(axis=0)
    assert col[Q].max() < col[K].min() * (1 + 1e-6)
    np.testing.assert_array_equal(Wo[~rows], W[~rows])
    assert np.all(Wo[rows][:, Q] == 0.0)
    D = np.outer(W[rows][:, Q] @ v[Q], v[K] / E[K]) / (1 + (v[K] ** 2 / E[K]).sum())
    d = np.sqrt(E + v * v)[K]
    e = np.linalg.norm((Wo[rows][:, K] - (W[rows][:, K] + D)) * d) / np.linalg.norm(D * d)
    kept = np.linalg.norm(W[rows][:, K] * d) / np.linalg.norm(D * d)
    print(f"  {e:.2e}, kept weights {kept:.2f} times what is added", flush=True)
    assert e <= 2.0 ** -19 + 2.0 ** -24 * kept


def test_structured_with_every_column_removed():
    from tests.gpu_util import gpu_prune
    c, b = 64, 200
    W, H32 = _layer(c, b, 2 * b, "f32", seed=2)
    Wg, Mg, info = gpu_prune(W, H32, mode="structured", p=0.5, alpha=0.5)
    assert info == 0
    gone = Mg.any(axis=1)
    assert gone.sum() == 32 and Mg[gone].all()
    np.testing.assert_array_equal(Wg[gone], 0.0)
    np.testing.assert_array_equal(Wg[~gone], W[~gone])
