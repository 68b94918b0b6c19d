"""GPU parity of the one-launch kernel for 32 tokens or fewer in which a workgroup owns its rows for all columns: token
counts around its paddings, one and two row tiles per workgroup, fewer blocks than waves, part of a last block, runs of
weak columns (more than four to a block, none, all of a block), zero points that are no small integers.

Bar: relative L2 error <= 1e-3, max-abs <= 1e-2 * rms(y), whole output and per token, as for the layout's other kernels."""
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


@pytest.mark.parametrize("d_in,d_out,bits,group,k,tokens", [
    (1024, 33, 3, 128, 8, 1), (1024, 64, 4, 0, 8, 4), (2048, 200, 3, 0, 20, 5), (640, 96, 4, 256, 6, 8), (1160, 40, 3, 128, 9, 9),
    (1000, 70, 4, 128, 7, 16), (1032, 31, 3, 256, 4, 17), (2048, 130, 4, 128, 21, 32), (100 * 8, 8250, 4, 128, 8, 16),
    (256, 16400, 3, 0, 3, 16), (512, 8300, 3, 128, 0, 31), (104, 40, 4, 0, 2, 3), (4096, 64, 3, 128, 300, 12)])
@pytest.mark.parametrize("zeros", ["integers", "any"])
def test_layers_match_oracle(env, d_in, d_out, bits, group, k, tokens, zeros):
    torch, B = env
    layer = make_layer(LayerSpec("few", d_in, d_out, bits, group, k, d_in + tokens))
    if zeros == "any":
        rng = np.random.default_rng(tokens)
        z = layer.zero.astype(np.float32) + rng.normal(0, 2, layer.zero.shape)
        z[rng.random(z.shape) < 0.05] = -2500.5
        layer.zero[:] = z.astype(np.float16)
    x = make_x(layer, tokens)
    print(f"{d_in} -> {d_out}, {bits} bit, group {group}, k {k}, {tokens} tokens, zero points: {zeros}", flush=True)
    lin = B.OwqLinear(layer, layout=TILE)
    y = lin(torch.from_numpy(x).cuda()).cpu().numpy()
    check(y, owq_ref.owq_linear_layer(layer, x), "few")
    lin.close()


@pytest.mark.parametrize("runs", [[(0, 128)], [(60, 70), (300, 309)], [(127, 129), (1020, 1024)], [(512, 640), (700, 701)]])
def test_runs_of_weak_columns(env, runs):
    torch, B = env
    idx = np.concatenate([np.arange(a, b) for a, b in runs]).astype(np.int32)
    layer = make_layer(LayerSpec("runs", 1024, 96, 4, 128, len(idx), 17))
    rng = np.random.default_rng(3)
    layer.codes[:] = rng.integers(0, 16, layer.codes.shape)
    layer.codes[:, idx] = 0
    layer.weak_idx[:] = idx
    x = make_x(layer, 13)
    x[:, idx] *= np.float16(20)
    lin = B.OwqLinear(layer, layout=TILE)
    check(lin(torch.from_numpy(x).cuda()).cpu().numpy(), owq_ref.owq_linear_layer(layer, x), runs)
    # what stands at the weak columns reaches the result through the weak weights only
    layer.weak_w[:] = 0
    B.owq_update_weak(lin.handle, layer.weak_w)
    a = lin(torch.from_numpy(x).cuda()).cpu().numpy()
    x[:, idx] = np.float16(30000)
    np.testing.assert_array_equal(a.view(np.uint16), lin(torch.from_numpy(x).cuda()).cpu().numpy().view(np.uint16))
    lin.close()


@pytest.mark.parametrize("d_in,d_out,bits,group,k,tokens", [(4736, 549, 4, 384, 30, 1), (4352, 1645, 4, 640, 9, 2), (7680, 2048, 3, 384, 20, 4),
                                                            (7680, 2048, 3, 384, 20, 16)])
def test_groups_that_no_other_kernel_takes(env, d_in, d_out, bits, group, k, tokens):
    # groups that are not 128 2^n: the kernel that spreads columns refuses them, so its cost must not count
    from launches import launches
    torch, B = env
    layer = make_layer(LayerSpec("groups", d_in, d_out, bits, group, k, d_in))
    x = make_x(layer, tokens)
    print(f"{d_in} -> {d_out}, {bits} bit, group {group}, {tokens} tokens", flush=True)
    lin = B.OwqLinear(layer, layout=TILE)
    xd, y = torch.from_numpy(x).cuda(), torch.empty((tokens, d_out), dtype=torch.float16, device="cuda")
    assert len(launches(torch, lambda: lin(xd, out=y))) == 1
    check(y.cpu().numpy(), owq_ref.owq_linear_layer(layer, x), "groups")
    lin.close()
