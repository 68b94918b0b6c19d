"""A launch shape asked for with owq_set_launch holds for every token count that the header names: the passes of a long
batch and the calls of 17 to 32 tokens, which the library would send to other kernels by itself, give the bits of the
shaped kernels, and a shape that does not fit the last pass is an error."""
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


def bits(t):
    return t.cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("shape", [(0, 2, 4, 0), (5, 0, 0, 0), (0, 0, 4, 0), (0, 0, 0, -1), (0, 0, 0, 3), (0, 3, 0, -1)])
def test_long_batches_run_in_passes_of_the_shape(env, shape):
    torch, B = env
    layer = make_layer(LayerSpec("long", 2048, 700, 3, 128, 20, 41))
    x = torch.from_numpy(make_x(layer, 64 + 64 + 9)).cuda()
    lin = B.OwqLinear(layer, layout=1)
    other = bits(lin(x))                                        # the library's choice: another kernel
    B.owq_set_launch(lin.handle, *shape)
    got = lin(x)
    passes = torch.cat([lin(x[i:i + 64].contiguous()) for i in range(0, 137, 64)])
    np.testing.assert_array_equal(bits(got), bits(passes))
    assert (bits(got) != other).any()
    rel, mx = owq_ref.parity_errors(got.cpu().numpy(), owq_ref.owq_linear_layer(layer, x.cpu().numpy()))
    assert rel <= 1e-3 and mx <= 1e-2, (rel, mx)
    B.owq_set_launch(lin.handle, 0, 0, 0, 0)                    # and the library chooses again
    np.testing.assert_array_equal(bits(lin(x)), other)
    lin.close()


@pytest.mark.parametrize("shape", [(0, 2, 4), (7, 0, 0)])
def test_calls_of_17_to_32_tokens_take_the_shaped_launches(env, shape):
    torch, B = env
    layer = make_layer(LayerSpec("mid", 2048, 700, 4, 0, 20, 42))
    x = torch.from_numpy(make_x(layer, 24)).cuda()
    lin = B.OwqLinear(layer, layout=1)
    B.owq_set_launch(lin.handle, *shape, -1)                    # the three launches for any number of tokens
    want = bits(lin(x))
    B.owq_set_launch(lin.handle, *shape, 0)
    np.testing.assert_array_equal(bits(lin(x)), want)
    rel, mx = owq_ref.parity_errors(lin(x).cpu().numpy(), owq_ref.owq_linear_layer(layer, x.cpu().numpy()))
    assert rel <= 1e-3 and mx <= 1e-2, (rel, mx)
    lin.close()


def test_a_last_pass_that_does_not_fit_is_an_error(env):
    # one range of 24 blocks for 32 tokens is more than a workgroup stages
    torch, B = env
    layer = make_layer(LayerSpec("nofit", 3072, 64, 3, 0, 4, 3))
    x = torch.from_numpy(make_x(layer, 64 + 32)).cuda()
    lin = B.OwqLinear(layer, layout=1)
    B.owq_set_launch(lin.handle, 0, 0, 0, 1)
    with pytest.raises(B.OwqError) as e:
        lin(x)
    assert e.value.status == B.OWQ_ERR_SHAPE
    lin.close()
