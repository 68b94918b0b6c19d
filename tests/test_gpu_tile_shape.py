"""The default work split of the tile layout's passes of 33 to 64 tokens: ranges are joined where workgroups have few steps or
an eighth of them is left out; everywhere else the whole chip is used, and the order of the partial sums follows."""
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
    (9216, 36864, 256, 0),        # 21 steps each: 247 would do, and save one workgroup in 28
    (36864, 9216, 252, 7),
    (13824, 5120, 240, 12),       # five steps: 11 ranges instead of 12 would save one in 12
    (5248, 11617, 242, 0),        # four steps
    (7000, 3333, 196, 14),        # two steps: 14 ranges instead of 18
])
def test_default_split(env, d_in, d_out, workgroups, splits):
    torch, B = env
    desc = B.make_desc(d_out, d_in, 3, 0, 16, layout=1)
    buf = torch.empty(B.owq_packed_bytes(desc), dtype=torch.uint8, device="cuda")
    handle = B.owq_open_packed(desc, buf.data_ptr(), buf.numel())
    info = B.owq_layer_info(handle)
    B.owq_free_layer(handle)
    assert (info.workgroups, info.row_splits) == (workgroups, splits)


@pytest.mark.parametrize("d_in,d_out", [(7000, 3333), (6528, 5000)])
def test_the_default_is_what_its_numbers_say(env, d_in, d_out):
    torch, B = env
    layer = make_layer(LayerSpec("split", d_in, d_out, 3, 0, 16, d_in))
    x = torch.from_numpy(make_x(layer, 40)).cuda()
    lin = B.OwqLinear(layer, layout=1)
    info = lin.info()
    got = lin(x).cpu().numpy()
    rows = np.unique(np.random.default_rng(1).integers(0, d_out, 100))
    want = owq_ref.owq_linear_ref(layer.codes[rows], layer.scale[rows], layer.zero[rows], 0, layer.weak_idx, layer.weak_w[rows],
                                  x.cpu().numpy())
    rel, mx = owq_ref.parity_errors(got[:, rows], want)
    assert rel <= 1e-3 and mx <= 1e-2, (rel, mx)
    # the same split asked for gives the same sums
    B.owq_set_launch(lin.handle, 0 if info.row_splits else info.workgroups, info.row_splits, 4, 0)
    np.testing.assert_array_equal(got.view(np.uint16), lin(x).cpu().numpy().view(np.uint16))
    lin.close()
