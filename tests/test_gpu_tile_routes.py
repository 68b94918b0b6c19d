"""Branches of the tile layout's kernels that calls of ordinary sizes do not reach: the exact (row, column) mapping of the
three launches, more than 256 weak columns in the one-launch kernel that owns its rows, its neighbour that spreads columns
at shapes the library would give to it, prompts that the scratch area holds only in parts, and prompts that run as two
launches with different column splits.

Bar where it is not bit-exact: relative L2 error <= 1e-3, max-abs <= 1e-2 * rms(y), whole output and per token."""
import numpy as np
import pytest

from oracle import owq_ref
from synth import LayerSpec, make_layer, make_x

pytestmark = pytest.mark.gpu
TILE = 1


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2306_02272_amd import binding
    binding.lib()
    torch.cuda.set_device(0)
    return torch, binding


def check(got, want, what):
    for g, w in [(got, want)] + list(zip(got, want)):
        rel, mx = owq_ref.parity_errors(g, w)
        assert rel <= 1e-3 and mx <= 1e-2, (what, rel, mx)


@pytest.mark.parametrize("bits,group", [(3, 0), (4, 0), (3, 128), (4, 256)])
@pytest.mark.parametrize("tokens", [33, 64])
def test_one_hot_probing_of_the_three_launches(env, bits, group, tokens):
    # x = e_j reads the effective matrix back: fp16(s*(q-z)) at dense positions, Ww at weak ones
    torch, B = env
    d_in, d_out, k = 640, 300, 9
    layer = make_layer(LayerSpec("onehot3", d_in, d_out, bits, group, k, 71 + bits + group))
    eye = np.eye(d_in, dtype=np.float16)
    want = owq_ref.to_fp16(owq_ref.owq_linear_layer(layer, eye)).view(np.uint16)
    lin = B.OwqLinear(layer, layout=TILE)
    B.owq_set_launch(lin.handle, 0, 0, 0, -1)
    xd = torch.from_numpy(eye).cuda()
    y = torch.empty((d_in, d_out), dtype=torch.float16, device="cuda")
    print(f"{bits} bit, group {group}, {tokens} tokens a call", flush=True)
    for j0 in range(0, d_in, tokens):
        lin(xd[j0:j0 + tokens], out=y[j0:j0 + tokens])
    np.testing.assert_array_equal(y.cpu().numpy().view(np.uint16), want)
    np.testing.assert_array_equal(lin(xd).cpu().numpy().view(np.uint16), want)       # one call, ten passes
    lin.close()


@pytest.mark.parametrize("d_in,d_out,bits,group,k,tokens", [
    (2048, 64, 3, 128, 300, 12), (2048, 64, 4, 128, 512, 4), (1024, 96, 4, 128, 400, 20), (1024, 70, 3, 0, 257, 16), (2048, 8300, 4, 0, 260, 31)])
def test_many_weak_columns_in_one_launch(env, d_in, d_out, bits, group, k, tokens):
    torch, B = env
    layer = make_layer(LayerSpec("manyweak", d_in, d_out, bits, group, k, k + tokens))
    x = make_x(layer, tokens)
    print(f"{d_in} -> {d_out}, {bits} bit, k {k}, {tokens} tokens", flush=True)
    lin = B.OwqLinear(layer, layout=TILE)
    y = lin(torch.from_numpy(x).cuda()).cpu().numpy()
    check(y, owq_ref.owq_linear_layer(layer, x), "one launch")
    lin.close()


@pytest.mark.parametrize("d_in,d_out,bits,group,k,tokens", [
    (1024, 96, 3, 0, 8, 16), (512, 64, 3, 0, 4, 1), (768, 600, 3, 0, 24, 5), (2048, 130, 4, 128, 16, 16), (256, 40, 3, 0, 200, 12),
    (1024, 64, 3, 0, 24, 3), (512, 1, 3, 0, 2, 3), (8192, 64, 4, 128, 82, 16)])
def test_columns_spread_over_workgroups(env, d_in, d_out, bits, group, k, tokens):
    # prefetch_depth 100: that kernel, with its own choice of ranges
    torch, B = env
    layer = make_layer(LayerSpec("spread", d_in, d_out, bits, group, k, d_in + tokens))
    x = make_x(layer, tokens)
    lin = B.OwqLinear(layer, layout=TILE)
    B.owq_set_launch(lin.handle, 0, 0, 0, 100)
    print(f"{d_in} -> {d_out}, {bits} bit, k {k}, {tokens} tokens", flush=True)
    check(lin(torch.from_numpy(x).cuda()).cpu().numpy(), owq_ref.owq_linear_layer(layer, x), "spread")
    lin.close()


@pytest.mark.parametrize("d_in,d_out,bits,group,k,tokens", [
    (1001, 20, 4, 128, 7, 700),      # the scratch area holds the copied rows of 192 tokens: 3 x 192 and 124
    (1001, 32, 3, 0, 7, 500),
    (100, 33, 3, 0, 3, 2000)])       # 512 tokens a pass
def test_prompts_beyond_the_scratch_area(env, d_in, d_out, bits, group, k, tokens):
    torch, B = env
    layer = make_layer(LayerSpec("parts", d_in, d_out, bits, group, k, tokens))
    x = make_x(layer, tokens)
    print(f"{d_in} -> {d_out}, {tokens} tokens", flush=True)
    lin = B.OwqLinear(layer, layout=TILE)
    check(lin(torch.from_numpy(x).cuda()).cpu().numpy(), owq_ref.owq_linear_layer(layer, x), "parts")
    lin.close()


def test_a_prompt_in_two_launches(env):
    # 32 row groups x 17 token tiles: 512 tiles fill the chip once, the 17th token tile runs by itself, its columns in four
    torch, B = env
    layer = make_layer(LayerSpec("two", 4096, 8000, 3, 128, 40, 72))
    x = make_x(layer, 1060)
    lin = B.OwqLinear(layer, layout=TILE)
    y = lin(torch.from_numpy(x).cuda()).cpu().numpy()
    rows = np.unique(np.concatenate([np.random.default_rng(2).integers(0, 8000, 150), [0, 255, 256, 7935, 7936, 7999]]))
    want = owq_ref.owq_linear_ref(layer.codes[rows], layer.scale[rows], layer.zero[rows], 128, layer.weak_idx, layer.weak_w[rows], x)
    check(y[:, rows], want, "two launches")
    lin.close()
