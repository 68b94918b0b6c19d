"""The 256-row x 64- and 128-token tiles for prompts against the fp64 CPU oracle, on layers that only they take (more weak
columns than the one-launch kernel's LDS holds) or that are large enough for them: last tiles that are nearly empty, odd
numbers of blocks, rows off the 16-byte grid, zero points that are no small integers, and step sizes that one block's
sums cannot be divided by (zero) or hardly (subnormal, the largest, negative).

Bar as for the other kernels of the layout: relative L2 error <= 1e-3, max-abs error <= 1e-2 rms, whole output and per token."""
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


def compare(env, layer, x, what, rows=300):
    torch, B = env
    lin = B.OwqLinear(layer, layout=1)
    got = lin(torch.from_numpy(x).cuda()).cpu().numpy()
    again = lin(torch.from_numpy(x).cuda()).cpu().numpy()
    np.testing.assert_array_equal(got.view(np.uint16), again.view(np.uint16))
    lin.close()
    d_out = layer.d_out
    pick = np.unique(np.concatenate([np.arange(max(0, d_out - 40), d_out),
                                     np.random.default_rng(1).integers(0, d_out, min(rows, d_out))]))
    want = owq_ref.owq_linear_ref(layer.codes[pick], layer.scale[pick], layer.zero[pick], layer.group_size, layer.weak_idx,
                                  layer.weak_w[pick], x)
    for g, w in [(got[:, pick], want)] + list(zip(got[:, pick], want)):
        rel, mx = owq_ref.parity_errors(g, w)
        assert rel <= 1e-3 and mx <= 1e-2, (what, rel, mx)


@pytest.mark.parametrize("d_in,d_out,bits,group,k,tokens", [
    (2048, 300, 3, 128, 1500, 65),        # split columns
    (1800, 257, 4, 0, 1450, 129),         # odd number of blocks and a part of one
    (1799, 70, 3, 128, 1400, 200),        # rows of x off the 16-byte grid
    (512, 8225, 3, 128, 5, 1153),         # tiles of 128 tokens, the last of one token
    (640, 8192, 4, 256, 0, 1090),
    (512, 8193, 4, 0, 9, 1100),
    (1600, 6401, 3, 128, 1400, 1000),
])
@pytest.mark.parametrize("zeros", ["integers", "any"])
def test_tiles_match_oracle(env, d_in, d_out, bits, group, k, tokens, zeros):
    layer = make_layer(LayerSpec("tiles", d_in, d_out, bits, group, k, d_in + d_out))
    if zeros == "any":
        rng = np.random.default_rng(5)
        rows = np.arange(d_out) // 256 % 2 == 0         # every other row group keeps its integers
        z = layer.zero.astype(np.float32) + np.where(rows[:, None], rng.normal(0, 2, layer.zero.shape), 0)
        z[rows & (rng.random(d_out) < 0.05)] = 1500.5
        layer.zero[:] = z.astype(np.float16)
    print(d_in, d_out, tokens, zeros, flush=True)
    compare(env, layer, make_x(layer, tokens), (d_in, d_out, tokens, zeros))


@pytest.mark.parametrize("d_in,d_out,bits,k,tokens", [(2048, 300, 3, 1500, 70), (1152, 8192, 4, 4, 1100)])
def test_step_sizes_of_neighbouring_groups_of_any_size(env, d_in, d_out, bits, k, tokens):
    layer = make_layer(LayerSpec("steps", d_in, d_out, bits, 128, k, 17))
    rng = np.random.default_rng(3)
    kind = rng.integers(0, 8, layer.scale.shape)
    s = layer.scale.astype(np.float64)
    s[kind == 0] *= -1
    s[kind == 1] = 3e-7                       # subnormal
    s[kind == 2] = 0.9
    s[(kind == 3) & (np.arange(d_out) // 256 % 2 == 0)[:, None]] = 0      # in every other row group
    layer.scale[:] = s.astype(np.float16)
    print(d_in, d_out, tokens, flush=True)
    compare(env, layer, make_x(layer, tokens), (d_in, d_out, tokens))


@pytest.mark.parametrize("bits,k,d_out,tokens", [(3, 1500, 300, 512), (4, 30, 8192, 1100)])
def test_one_column_by_itself_is_exact(env, bits, k, d_out, tokens):
    # x = a column of the identity in 24 groups: s (q - z) has 15 bits at most, so often a tie of fp16. 23 ratios, each
    # multiplication off by half a unit of the last place and all ratios together by one or two, leave less than the
    # 16 units within which the result is settled.
    torch, B = env
    layer = make_layer(LayerSpec("columns", 3072, d_out, bits, 128, k, 23))
    cols = np.random.default_rng(9).integers(0, 3072, tokens)
    x = np.zeros((tokens, 3072), np.float16)
    x[np.arange(tokens), cols] = 1
    lin = B.OwqLinear(layer, layout=1)
    got = lin(torch.from_numpy(x).cuda()).cpu().numpy()
    lin.close()
    pick = np.random.default_rng(2).integers(0, d_out, 200)
    want = owq_ref.to_fp16(owq_ref.owq_linear_ref(layer.codes[pick], layer.scale[pick], layer.zero[pick], layer.group_size,
                                                  layer.weak_idx, layer.weak_w[pick], x))
    np.testing.assert_array_equal(got[:, pick].view(np.uint16), want.view(np.uint16))
