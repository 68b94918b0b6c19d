"""Configuration search by diagonals: ranges of which a diagonal has one step size in the first half of its points and another
one in the second, which is what the two lanes of a diagonal see.  Such ranges are a handful in 10^5, and few of their groups
have their least error there, so both are looked for on the host: ends whose binary32 widths straddle the middle between two
binary16 step sizes between the halves (diagonals of two and three points among them), and weights between these ends whose
best grid point, by the oracle's arithmetic, has a step size that the other half does not.

Every output is compared with the general way bit for bit (the same rows in calls of fewer groups) and the choice with the
oracle's errors: binary32 sums of binary32 residuals, 1e-5 of the least error, or 2^-22 of the squared weights."""
import numpy as np
import pytest

from oracle import search

pytestmark = pytest.mark.gpu
F32 = np.float32
COLS = 4096


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_02272_amd import binding
    binding.lib()
    torch.cuda.set_device(0)
    return torch, binding


def step_sizes(lo, hi, bits, n, shrink):
    """Step sizes as bit patterns [range][i][j] of the ranges lo, hi (binary32 arrays): the operations of search.candidate."""
    cut = search.cut_fractions(n, shrink)[None] * (hi - lo).astype(F32)[:, None]
    lo_i, hi_j = lo[:, None] + cut, hi[:, None] - cut
    s = (hi_j[:, None, :] - lo_i[:, :, None]) / F32((1 << bits) - 1)
    assert s.dtype == F32
    return np.maximum(s, F32(2.0 ** -14)).astype(np.float16).view(np.uint16)


def halves(n, d):
    """Lower-end indices of the two halves of diagonal d."""
    first, last = max(0, d - (n - 1)), min(d, n - 1)
    mid = first + (last - first + 2) // 2
    return np.arange(first, mid), np.arange(mid, last + 1)


def split_ranges(bits, n, shrink, rng, draws):
    """(lo, hi, diagonal) of ranges with a diagonal of one step size per half, not the same, and one each on all others."""
    found = []
    for _ in range(draws):
        lo = -np.abs(rng.normal(0.1, 0.06, 20000)).astype(np.float16).astype(F32)
        hi = np.abs(rng.normal(0.1, 0.06, 20000)).astype(np.float16).astype(F32)
        s = step_sizes(lo, hi, bits, n, shrink)
        one = np.ones((len(lo), 2 * n - 1), dtype=bool)
        two = np.zeros_like(one)
        for d in range(2 * n - 1):
            a, b = halves(n, d)
            sa = s[:, a, d - a]
            sb = s[:, b, d - b] if b.size else sa[:, -1:]
            each = (sa == sa[:, :1]).all(1) & (sb == sb[:, :1]).all(1)
            one[:, d] = each & (sa[:, 0] == sb[:, 0])
            two[:, d] = each & (sa[:, 0] != sb[:, 0])
        found += [(lo[r], hi[r], int(np.argmax(two[r]))) for r in np.nonzero((one | two).all(1) & (two.sum(1) == 1))[0]]
    return found


def groups_of(lo, hi, d, bits, n, shrink, group, rng, draws):
    """Groups of weights with these ends whose least error is on diagonal d: near the levels of a grid point of it, which the
    ends need not be."""
    qmax = F32((1 << bits) - 1)
    cut = search.cut_fractions(n, shrink)
    w = np.empty((draws, group), dtype=np.float16)
    for k, i in enumerate(rng.choice(np.concatenate(halves(n, d)), draws)):
        s, _, z = search.candidate(lo, hi, cut[i], cut[d - i], int(qmax))
        w[k] = np.clip(s * (rng.integers(0, int(qmax) + 1, group) - z + rng.uniform(-0.3, 0.3, group)), lo, hi)
    w[:, 5], w[:, 77] = lo, hi
    w32 = w.astype(F32)
    points = {}
    for i in range(n):
        for j in range(n):
            points.setdefault(tuple(search.candidate(lo, hi, cut[i], cut[j], int(qmax))), []).append((i, j))
    errs = []
    for s, inv, z in points:
        q = np.clip(np.rint(w32 * F32(inv)) + F32(z), F32(0), qmax)
        errs.append(((w.astype(np.float64) - np.float64(s) * (q.astype(np.float64) - np.float64(z))) ** 2).sum(1))
    best = np.argmin(np.stack(errs), axis=0)
    on = [all(i + j == d for i, j in ids) for ids in points.values()]
    return w[np.array(on)[best]]


@pytest.mark.parametrize("bits,n,shrink,group,draws", [
    (4, 12, 0.294, 128, 2), (4, 12, 0.382, 1024, 20), (3, 16, 0.382, 512, 8), (3, 15, 0.31, 256, 20), (3, 14, 0.4, 1024, 20)])
def test_halves_of_a_diagonal_with_a_step_size_each(env, bits, n, shrink, group, draws):
    torch, B = env
    rng = np.random.default_rng(1000 * n + bits)
    ranges = split_ranges(bits, n, shrink, rng, draws)
    if shrink == 0.294:                            # two points, one zero point, a step size each
        ranges.insert(0, (F32(-0.046234130859375), F32(0.06573486328125), 1))
    assert len(ranges) >= 4
    hard = np.concatenate([groups_of(lo, hi, d, bits, n, shrink, group, rng, 60) for lo, hi, d in ranges])
    print(f"{bits} bit, {n} points, {shrink}, groups of {group}: {len(ranges)} ranges, diagonals {sorted({r[2] for r in ranges})}, "
          f"{len(hard)} groups", flush=True)
    assert len(hard) >= 50
    units = 16384 * max(1, 256 // group)           # 16384 groups, 4 Mi weights: by diagonals
    rows = units * group // COLS
    w = rng.normal(0, 0.02, (units, group)).astype(np.float16)
    at = rng.permutation(units)[:units // 2]
    w[at] = hard[np.arange(len(at)) % len(hard)]
    wd = torch.from_numpy(w.reshape(rows, COLS)).cuda()
    whole = B.search_config(wd, None, bits, group, n, n, shrink)
    parts = [B.search_config(wd[r:r + 500].contiguous(), None, bits, group, n, n, shrink) for r in range(0, rows, 500)]
    choice = whole[4].cpu().numpy().reshape(-1)
    wrong = {}
    for name, got, want in zip(("scale", "zero", "codes", "err", "choice"), whole, zip(*parts)):
        got, want = (t.cpu().numpy().reshape(units, -1).view(np.uint8) for t in (got, torch.cat(list(want))))
        wrong[name] = int((got != want).any(1).sum())
    assert not any(wrong.values()), wrong
    for i in range(0, len(hard), max(1, len(hard) // 60)):
        es = search.candidate_errors(hard[i], np.ones(group, dtype=bool), bits, n, n, shrink)
        assert es[choice[at[i]]] <= es.min() * (1 + 1e-5) + 2.0 ** -44 * float((hard[i].astype(np.float64) ** 2).sum()), i
