"""The 256-row x 64- and 128-token tiles for prompts against the fp64 CPU oracle, on layers that only they take (more weak
columns than the one-launch kernel's LDS holds) or that are large enough for them: last tiles that are nearly empty, odd
numbers of blocks, rows off the 16-byte grid, zero points that are no small integers, and step sizes of any size and sign
in neighbouring groups (zero, subnormal, large).

Bar as for the other kernels of the layout: relative L2 error <= 1e-3, max-abs error <= 1e-2 rms, whole output and per token."""
import numpy as np
import pytest

from launches import launches
from oracle import owq_ref
from synth import Layer, LayerSpec, make_layer, make_x

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


def compare(env, layer, x, what, rows=300, rounding=False, eight=None):
    torch, B = env
    lin = B.OwqLinear(layer, layout=1)
    if eight is not None:                  # workgroups of eight waves, 0: none
        xd, y = torch.from_numpy(x).cuda(), torch.empty((len(x), layer.d_out), dtype=torch.float16, device="cuda")
        assert sum(n for n, threads in launches(torch, lambda: lin(xd, out=y)) if threads == 512) == eight, what
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
        # rounding: rows of large zero points can be more than 20 rms, whose rounding to fp16 alone is 2^-11 of them
        top = max(1e-2, 2.0 ** -11 * np.abs(w).max() / np.sqrt(np.mean(np.square(w))) + 2e-3) if rounding else 1e-2
        assert rel <= 1e-3 and mx <= top, (what, rel, mx)


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
def test_tiles_match_oracle(env, d_in, d_out, bits, group, k, tokens, zeros, rounding=False, eight=None):
    layer = make_layer(LayerSpec("tiles", d_in, d_out, bits, group, k, d_in + d_out))
    if zeros == "any":
        rng = np.random.default_rng(5)
        rows = np.arange(d_out) // 256 % 2 == 0         # every other row group keeps its integers
        z = layer.zero.astype(np.float32) + np.where(rows[:, None], rng.normal(0, 2, layer.zero.shape), 0)
        z[rows & (rng.random(d_out) < 0.05)] = 1500.5
        layer.zero[:] = z.astype(np.float16)
    print(d_in, d_out, tokens, zeros, flush=True)
    compare(env, layer, make_x(layer, tokens), (d_in, d_out, tokens, zeros), rounding=rounding, eight=eight)


# Workgroups of eight waves, whose halves take half the columns each, and how many of them: no column ranges beside, an odd number
# of blocks and a last tile whose second 64 tokens do not exist; a round of whole tiles and the others in five ranges, rows of x
# off the 16-byte grid; the same where the copied rows leave no room for partial results, four waves; two ranges of all tiles;
# one scale per row, a round of whole tiles and the others in four ranges.
@pytest.mark.parametrize("d_in,d_out,bits,group,k,tokens,eight", [
    (8056, 3300, 3, 128, 40, 1950, 13 * 16), (4100, 6600, 4, 128, 40, 1300, 256 + 5 * 30), (4100, 5120, 4, 128, 40, 2000, 0),
    (13824, 5100, 4, 256, 300, 590, 2 * 100), (8192, 5120, 3, 0, 9, 2040, 256 + 4 * 64)])
@pytest.mark.parametrize("zeros", ["integers", "any"])
def test_tiles_of_two_halves_match_oracle(env, d_in, d_out, bits, group, k, tokens, eight, zeros):
    test_tiles_match_oracle(env, d_in, d_out, bits, group, k, tokens, zeros, rounding=True, eight=eight)


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
    # x = a column of the identity in 24 groups: s (q - z) has 15 bits at most, so often a tie of fp16, and has to come out as
    # it is, rounded once.
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


@pytest.mark.parametrize("d_in,bits,d_out,tokens", [(16384, 3, 8192, 2048), (36864, 4, 8192, 2048)])
def test_one_column_by_itself_is_exact_whatever_the_number_of_groups(env, d_in, bits, d_out, tokens):
    # As above with 128 and 288 groups, all in one workgroup: the others add exact zeros to the column's and nothing else.
    torch, B = env
    rng = np.random.default_rng(4)
    groups = d_in // 128
    layer = Layer(LayerSpec("manygroups", d_in, d_out, bits, 128, 0, 0), rng.integers(0, 1 << bits, (d_out, d_in), dtype=np.uint8),
                  rng.uniform(0.001, 0.01, (d_out, groups)).astype(np.float16),
                  rng.integers(0, 1 << bits, (d_out, groups)).astype(np.float16), np.zeros(0, np.int32), np.zeros((d_out, 0), np.float16))
    cols = np.arange(tokens) % 512
    x = torch.zeros((tokens, d_in), dtype=torch.float16, device="cuda")
    x[torch.arange(tokens), torch.from_numpy(cols).cuda()] = torch.from_numpy(rng.choice([0.5, 1, 2, 3, 5, 7], tokens)).half().cuda()
    print(d_in, d_out, tokens, flush=True)
    lin = B.OwqLinear(layer, layout=1)
    got = lin(x).cpu().numpy()
    lin.close()
    g = cols // 128
    want = layer.scale[:, g].astype(np.float64) * (layer.codes[:, cols].astype(np.float64) - layer.zero[:, g]) * x.amax(1).cpu().numpy()
    np.testing.assert_array_equal(got.view(np.uint16), owq_ref.to_fp16(want.T + 0.0).view(np.uint16))


@pytest.mark.parametrize("group", [0, 128, 256])
def test_exact_sums_are_rounded_once(env, group):
    # Step sizes that are powers of two and small whole x: every sum is an exact binary32 number, with more than the 19 bits
    # that decide an fp16 number and its ties, so y has to be that sum rounded once.
    torch, B = env
    layer = make_layer(LayerSpec("powers", 2048, 8192, 4, group, 0, 31))
    rng = np.random.default_rng(6)
    layer.scale[:] = np.ldexp(1.0, rng.integers(-4, 5, layer.scale.shape)).astype(np.float16)
    x = rng.integers(-8, 9, (1100, 2048)).astype(np.float16)
    x[:, 1024:] = 0
    print("groups of", group, flush=True)
    lin = B.OwqLinear(layer, layout=1)
    got = lin(torch.from_numpy(x).cuda()).cpu().numpy()
    lin.close()
    want = owq_ref.to_fp16(owq_ref.owq_linear_ref(layer.codes, layer.scale, layer.zero, layer.group_size, layer.weak_idx,
                                                  layer.weak_w, x))
    np.testing.assert_array_equal(got.view(np.uint16), want.view(np.uint16))


@pytest.mark.parametrize("bits,group,tokens", [(3, 128, 1100), (4, 128, 100), (4, 256, 1100), (3, 0, 1100), (4, 0, 100)])
def test_zero_points_at_the_edge_of_what_the_unpack_takes(env, bits, group, tokens):
    # Integers of up to 1024 leave with the codes, others by a rest, chosen by 256 rows: row groups with 1024 and -1024, with 1025,
    # with 241 and with half-integers, a column of the identity (times 1 or 3) each: at most 24 bits, so exact until y is rounded.
    torch, B = env
    layer = make_layer(LayerSpec("edge", 640, 8200, bits, group, 0, 41))
    rng = np.random.default_rng(8)
    rows = np.arange(8200) // 256 % 5
    for kind, z in enumerate([1024, 1025, 241, 240.5]):
        pick = (rows == kind)[:, None] & (rng.random(layer.zero.shape) < 0.3)
        layer.zero[pick] = z
        if kind < 2:
            layer.zero[pick & (rng.random(layer.zero.shape) < 0.5)] = -z
    cols = np.random.default_rng(1).integers(0, 640, tokens)
    x = np.zeros((tokens, 640), np.float16)
    x[np.arange(tokens), cols] = rng.choice([1, 3], tokens)
    print(bits, "bit, groups of", group, tokens, "tokens", flush=True)
    lin = B.OwqLinear(layer, layout=1)
    got = lin(torch.from_numpy(x).cuda()).cpu().numpy()
    lin.close()
    g = cols // group if group else np.zeros(tokens, int)
    want = layer.scale[:, g].astype(np.float64) * (layer.codes[:, cols].astype(np.float64) - layer.zero[:, g]) * x.max(1).astype(np.float64)
    np.testing.assert_array_equal(got.view(np.uint16), owq_ref.to_fp16(want.T + 0.0).view(np.uint16))
