"""The configuration search rules grid points out by bounds from a histogram: every group must still get the grid point
with the least error.  Sizes where the kernel changes (groups a wave or four waves hold, runs of columns per lane,
rows off their grid, the last short group) and weights for which bounds are weak or useless: on a quantiser grid (error
zero), far from zero, with a step size at its least value, nearly all equal.

The oracle's errors are binary64 sums; the kernel ranks binary32 sums of binary32 residuals, so a group may keep a grid
point whose error is within 1e-5 of the least (a hundred times 2^-24, sums of at most a few hundred terms per lane), or,
where errors vanish against the weights, within what binary32 residuals can show (2^-22 of the squared weights)."""
import numpy as np
import pytest

from oracle import search

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_02272_amd import binding
    binding.lib()
    torch.cuda.set_device(0)
    return torch, binding


def weights(kind, rows, cols, rng):
    w = rng.normal(0, 0.02, (rows, cols))
    if kind == "grid":
        w = rng.integers(-3, 5, (rows, cols)) * 0.0625
    elif kind == "offset":
        w = w * 0.1 + 3.0
    elif kind == "least_step":
        w = w * 1e-3
    elif kind == "sparse":
        w = np.where(rng.random((rows, cols)) < 0.97, 0.0, w)
    elif kind == "tail":
        w = np.where(rng.random((rows, cols)) < 0.01, 8 * w, w)
    return w.astype(np.float16)


@pytest.mark.parametrize("d_in,group", [(100, 0), (129, 128), (300, 128), (512, 256), (1024, 512), (1000, 0), (1025, 0), (2048, 0), (2052, 0),
                                        (4097, 0), (6144, 0), (6152, 0), (12289, 0), (16384, 0), (16385, 0)])
@pytest.mark.parametrize("kind", ["normal", "grid", "offset", "least_step", "sparse", "tail"])
def test_every_group_gets_the_least_error(env, d_in, group, kind):
    torch, B = env
    rng = np.random.default_rng(d_in + group)
    rows = 2 if d_in > 2048 else 5
    n_lo, n_hi, bits = (16, 16, 3) if kind in ("normal", "grid", "least_step") else (7, 9, 4)
    if d_in > 4096:
        n_lo, n_hi = 5, 6
    w = weights(kind, rows, d_in, rng)
    idx = np.sort(rng.choice(d_in, max(1, d_in // 100), replace=False)).astype(np.int32)
    keep = np.ones(d_in, dtype=bool)
    keep[idx] = False
    print(f"d_in {d_in} group {group} {kind}", flush=True)
    scale, zero, codes, err, choice = (t.cpu().numpy() for t in B.search_config(torch.from_numpy(w).cuda(), torch.from_numpy(idx).cuda(),
                                                                                 bits, group, n_lo, n_hi, 0.4))
    g = group or d_in
    for r in range(rows):
        for gi in range(err.shape[1]):
            sl = slice(gi * g, min(d_in, gi * g + g))
            es = search.candidate_errors(w[r, sl], keep[sl], bits, n_lo, n_hi, 0.4)
            if not np.isfinite(es).any():          # nothing to search
                assert choice[r, gi] == 0 and err[r, gi] == 0 and not codes[r, sl].any()
                continue
            kept = w[r, sl].astype(np.float64)[keep[sl]]
            floor = 2.0 ** -44 * float((kept ** 2).sum())
            assert es[choice[r, gi]] <= es.min() * (1 + 1e-5) + floor, (r, gi, choice[r, gi], int(es.argmin()))
            assert abs(err[r, gi] - es[choice[r, gi]]) <= 1e-4 * es[choice[r, gi]] + floor
            s, z, q, _, _ = search.search_group(w[r, sl], keep[sl], bits, n_lo, n_hi, 0.4) if choice[r, gi] == es.argmin() else [None] * 5
            if s is not None:
                assert scale[r, gi] == s and zero[r, gi] == z
                np.testing.assert_array_equal(codes[r, sl], q)


def test_a_group_that_holds_no_numbers_leaves_its_neighbours_alone(env):
    torch, B = env
    rng = np.random.default_rng(9)
    w = weights("normal", 4, 512, rng)
    bad = w.copy()
    bad[1, 130], bad[2, 260], bad[3, 3] = np.nan, np.inf, -np.inf
    a, b = ([t.cpu().numpy() for t in B.search_config(torch.from_numpy(v).cuda(), None, 3, 128, 16, 16, 0.4)] for v in (w, bad))
    same = np.ones((4, 4), dtype=bool)
    same[1, 1] = same[2, 2] = same[3, 0] = False
    for x, y in ((a[0], b[0]), (a[1], b[1]), (a[3], b[3]), (a[4], b[4])):
        np.testing.assert_array_equal(x[same], y[same])
    np.testing.assert_array_equal(a[2].reshape(4, 4, 128)[same], b[2].reshape(4, 4, 128)[same])
