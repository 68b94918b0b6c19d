"""Configuration search of groups so narrow that some or all step sizes sit at their least value 2^-14: bounds rule little
out there, and many grid points have the same step size and zero point, of which one stands for all.  Every group must
get the least error and the lowest grid point that has it; bar as in test_gpu_search_bounds."""
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


@pytest.mark.parametrize("d_in,group", [(300, 128), (512, 256), (1000, 0), (1500, 0), (5120, 0)])
@pytest.mark.parametrize("std", [2e-7, 4e-5, 1e-4, 4e-4])
@pytest.mark.parametrize("bits", [3, 4])
def test_every_group_gets_the_least_error(env, d_in, group, std, bits):
    torch, B = env
    rng = np.random.default_rng(d_in + bits)
    rows, n_lo, n_hi = 3, 16, 16 if d_in < 1500 else 7
    w = rng.normal(0, std, (rows, d_in)).astype(np.float16)
    keep = np.ones(d_in, dtype=bool)
    idx = np.arange(5, d_in, 97, dtype=np.int32)
    keep[idx] = False
    print(f"d_in {d_in} group {group} std {std} bits {bits}", flush=True)
    scale, zero, codes, err, choice = (t.cpu().numpy() for t in B.search_config(torch.from_numpy(w).cuda(), torch.from_numpy(idx).cuda(),
                                                                                 bits, group, n_lo, n_hi, 0.4))
    g = group or d_in
    for r in range(rows):
        for gi in range(err.shape[1]):
            sl = slice(gi * g, min(d_in, gi * g + g))
            es = search.candidate_errors(w[r, sl], keep[sl], bits, n_lo, n_hi, 0.4)
            floor = 2.0 ** -44 * float((w[r, sl].astype(np.float64)[keep[sl]] ** 2).sum())
            assert es[choice[r, gi]] <= es.min() * (1 + 1e-5) + floor, (r, gi, choice[r, gi], int(es.argmin()))
            # no lower grid point has the same step size and zero point, hence the same error
            assert not (es[:choice[r, gi]] == es[choice[r, gi]]).any(), (r, gi, choice[r, gi])
            assert abs(err[r, gi] - es[choice[r, gi]]) <= 1e-4 * es[choice[r, gi]] + floor
