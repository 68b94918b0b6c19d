"""Configuration search of many groups on a square grid: the kernel that takes the grid by diagonals, and the one that takes
what is left to the general way, against the general way alone.

The same rows in calls of fewer groups take the general kernel, which test_gpu_search*.py compare with the oracle; both end
in the same operations on the same weights, so every output has to be the same bits, the errors among them.  Weights for
which diagonals are cut short or useless: far from zero (zero points beyond the levels), step sizes at their least value,
nearly all equal, on a grid (errors of zero, ties), no numbers; cuts at which the width of a diagonal lies halfway between
two step sizes (0.375 of 16: 7/8 of the range, a seventh of which is an eighth); short last groups and rows off the grid of
the lanes' loads."""
import numpy as np
import pytest

from launches import launches
from oracle import search
from test_gpu_search_bounds import weights

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


KINDS = ("normal", "grid", "offset", "least_step", "sparse", "tail", "nan")


@pytest.mark.parametrize("rows,cols,group,bits,n,shrink", [
    (1100, 4096, 128, 3, 16, 0.4), (1100, 4096, 128, 4, 16, 0.45), (1400, 3000, 128, 3, 12, 0.3), (2100, 2049, 256, 4, 16, 0.375),
    (2100, 2049, 256, 3, 16, 0.375), (2100, 4096, 512, 3, 13, 0.25), (2100, 4096, 512, 4, 16, 0.1), (4200, 4000, 1024, 3, 16, 0.4),
    (4200, 4000, 1024, 4, 12, 0.45), (1100, 4096, 128, 4, 16, 0.44), (4200, 4000, 1024, 4, 12, 0.44), (2100, 2049, 256, 3, 13, 0.45)])
def test_same_as_in_calls_of_fewer_groups(env, rows, cols, group, bits, n, shrink):
    torch, B = env
    assert rows * -(-cols // group) >= 16384 and rows * cols >= 4 << 20      # where the library takes diagonals
    rng = np.random.default_rng(rows + group + bits)
    per = -(-rows // len(KINDS))
    w = np.concatenate([weights(kind, per, cols, rng) for kind in KINDS])[:rows]
    m = rng.random(w[-per // 2:].shape)
    w[-per // 2:][m < 5e-4] = np.nan
    w[-per // 2:][m > 1 - 5e-4] = np.inf
    idx = torch.from_numpy(np.sort(rng.choice(cols, cols // 100, replace=False)).astype(np.int32)).cuda()
    wd = torch.from_numpy(w).cuda()
    whole = B.search_config(wd, idx, bits, group, n, n, shrink)
    # from 0.45 on at 4 bits zero points of a diagonal's half are further apart than a lane takes: the general kernel alone
    assert len(launches(torch, lambda: B.search_config(wd, idx, bits, group, n, n, shrink))) == (1 if bits == 4 and shrink >= 0.45 else 2)
    cut = 500 if group < 1024 else 900
    assert cut * cols < 4 << 20
    parts = [B.search_config(wd[r:r + cut].contiguous(), idx, bits, group, n, n, shrink) for r in range(0, rows, cut)]
    for name, got, want in zip(("scale", "zero", "codes", "err", "choice"), whole, zip(*parts)):
        got, want = got.cpu().numpy(), torch.cat(list(want)).cpu().numpy()
        same = got.view(np.uint8).reshape(rows, -1) == want.view(np.uint8).reshape(rows, -1)
        assert same.all(), (name, np.unique(np.nonzero(~same)[0])[:8])
    # and a few groups of each kind against the oracle itself
    keep_all = np.ones(cols, dtype=bool)
    keep_all[idx.cpu().numpy()] = False
    err, choice = whole[3].cpu().numpy(), whole[4].cpu().numpy()
    for r in range(3, rows - per // 2, per):
        for gi in (0, err.shape[1] - 1):
            sl = slice(gi * group, min(cols, gi * group + group))
            es = search.candidate_errors(w[r, sl], keep_all[sl], bits, n, n, shrink)
            kept = w[r, sl].astype(np.float64)[keep_all[sl]]
            if np.isfinite(es).any():
                # binary32 sums of binary32 residuals: 1e-5 of the least error, or 2^-22 of the squared weights
                assert es[choice[r, gi]] <= es.min() * (1 + 1e-5) + 2.0 ** -44 * float((kept ** 2).sum()), (r, gi)
