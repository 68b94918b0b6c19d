"""The default work split of the tile layout's passes of 33 to 64 tokens: ranges are joined only where that leaves an
eighth or more of the workgroups out; everywhere else the whole chip is used, and the order of the partial sums follows."""
import numpy as np
import pytest

from oracle import owq_ref
from synth import LayerSpec, make_layer, make_x

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


@pytest.mark.parametrize("d_in,d_out,workgroups,splits", [
    (32000, 1000, 256, 64),       # 4 row groups x 125 steps: 63 ranges of two steps would save one in 64
    (6400, 5120, 256, 0),         # 20 x 25 steps in equal ranges: 250 would save one in 43
    (7000, 3333, 196, 14),        # 14 x 28 steps: 14 ranges of two steps instead of 18 save two ninths
])
def test_default_split(env, d_in, d_out, workgroups, splits):
    torch, B = env
    layer = make_layer(LayerSpec("split", d_in, d_out, 3, 0, 16, d_in))
    x = torch.from_numpy(make_x(layer, 40)).cuda()
    lin = B.OwqLinear(layer, layout=1)
    info = lin.info()
    assert (info.workgroups, info.row_splits) == (workgroups, splits)
    got = lin(x).cpu().numpy()
    rows = np.unique(np.random.default_rng(1).integers(0, d_out, 100))
    want = owq_ref.owq_linear_ref(layer.codes[rows], layer.scale[rows], layer.zero[rows], 0, layer.weak_idx, layer.weak_w[rows],
                                  x.cpu().numpy())
    rel, mx = owq_ref.parity_errors(got[:, rows], want)
    assert rel <= 1e-3 and mx <= 1e-2, (rel, mx)
    # the same split asked for gives the same sums
    B.owq_set_launch(lin.handle, 0 if splits else workgroups, splits, 4, 0)
    np.testing.assert_array_equal(got.view(np.uint16), lin(x).cpu().numpy().view(np.uint16))
    lin.close()
