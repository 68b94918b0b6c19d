"""Backward of the dense part where its product's ranges of rows and its zero points can go wrong: rows that are no
multiple of a step of 128, ranges with an empty second half, one row tile, zero points that are fractions or beyond
what leaves with the unpack constant.  Bar as in test_gpu_backward: relative L2 error <= 1e-3, max-abs <= 1e-2 rms."""
import numpy as np
import pytest

from oracle import backward, owq_ref
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


@pytest.mark.parametrize("d_in,d_out,bits,group,k,tokens", [
    (256, 1, 3, 0, 4, 3), (256, 32, 4, 128, 4, 40), (300, 33, 3, 128, 9, 130), (512, 129, 4, 256, 5, 128),
    (1000, 260, 3, 0, 7, 65), (640, 999, 4, 128, 40, 257), (128, 1500, 3, 128, 3, 520), (768, 640, 4, 0, 200, 100)])
@pytest.mark.parametrize("zeros", ["integers", "any"])
def test_rows_and_zero_points(env, d_in, d_out, bits, group, k, tokens, zeros):
    torch, B = env
    layer = make_layer(LayerSpec("bwd", d_in, d_out, bits, group, k, d_in + d_out))
    rng = np.random.default_rng(d_out)
    if zeros == "any":
        z = layer.zero.astype(np.float32) + rng.normal(0, 2, layer.zero.shape)
        z[rng.random(z.shape) < 0.02] = 1100.5
        layer.zero[:] = z.astype(np.float16)
    x = make_x(layer, tokens)
    dy = rng.normal(0, 0.05, (tokens, d_out)).astype(np.float16)
    print(f"{d_in} -> {d_out}, {bits} bit, group {group}, k {k}, {tokens} tokens, zero points: {zeros}", flush=True)
    lin = B.OwqLinear(layer, layout=1)
    dx, dww = lin.backward(torch.from_numpy(dy).cuda(), torch.from_numpy(x).cuda())
    want_dx, want_dww = backward.owq_backward_ref(layer.codes, layer.scale, layer.zero, group, layer.weak_idx, layer.weak_w, x, dy)
    rel, mx = owq_ref.parity_errors(dx.cpu().numpy(), want_dx)
    assert rel <= 1e-3 and mx <= 1e-2, (rel, mx)
    rel, _ = owq_ref.parity_errors(dww.cpu().numpy(), want_dww)
    assert rel <= 1e-5, rel
    lin.close()


@pytest.mark.parametrize("lo,hi,grad", [(6e-8, 2e-6, 300.0), (20.0, 100.0, 1e-4), (0.3, 1.0, 2e-5)])
@pytest.mark.parametrize("zeros", ["integers", "any"])
def test_step_sizes_and_gradients_of_any_size(env, lo, hi, grad, zeros):
    # s (q - z) is rounded to fp16 by itself, with a relative error of 2^-11 at most also where s is subnormal, and dy is
    # not scaled: the same bar holds, dx being a normal number in all of these.
    torch, B = env
    layer = make_layer(LayerSpec("bwds", 600, 1000, 4, 128, 8, 3))
    rng = np.random.default_rng(11)
    layer.scale[:] = (rng.uniform(lo, hi, layer.scale.shape) * rng.choice([-1, 1], layer.scale.shape)).astype(np.float16)
    if zeros == "any":
        layer.zero[:] = (layer.zero.astype(np.float32) + rng.normal(0, 2, layer.zero.shape)).astype(np.float16)
    layer.weak_w[:] = 0
    x = make_x(layer, 150)
    dy = rng.normal(0, grad, (150, 1000)).astype(np.float16)
    print(f"step sizes {lo} to {hi}, gradients {grad}, zero points: {zeros}", flush=True)
    lin = B.OwqLinear(layer, layout=1)
    dx, _ = lin.backward(torch.from_numpy(dy).cuda(), torch.from_numpy(x).cuda())
    want, _ = backward.owq_backward_ref(layer.codes, layer.scale, layer.zero, 128, layer.weak_idx, layer.weak_w, x, dy)
    keep = np.ones(600, bool)
    keep[layer.weak_idx] = False
    rel, mx = owq_ref.parity_errors(dx.cpu().numpy()[:, keep], want[:, keep])
    assert rel <= 1e-3 and mx <= 1e-2, (rel, mx)
    lin.close()


@pytest.mark.parametrize("d_in,d_out,bits,group,k,tokens", [
    (4100, 40, 3, 128, 33, 2000),         # one range of rows, two sets of launches, columns off the 8-column grid
    (4099, 64, 4, 0, 0, 129),             # odd rows of dx, no weak columns, a pass of one token
    (8192, 260, 4, 128, 64, 300)])
def test_dx_stored_by_the_product(env, d_in, d_out, bits, group, k, tokens):
    torch, B = env
    layer = make_layer(LayerSpec("bwd1", d_in, d_out, bits, group, k, d_in))
    x = make_x(layer, tokens)
    dy = np.random.default_rng(d_in).normal(0, 0.05, (tokens, d_out)).astype(np.float16)
    print(f"{d_in} -> {d_out}, {tokens} tokens", flush=True)
    lin = B.OwqLinear(layer, layout=1)
    guard = torch.full((tokens + 1, d_in), 7.0, dtype=torch.float16, device="cuda")
    dyt, xt = torch.from_numpy(dy).cuda(), torch.from_numpy(x).cuda()
    ws = torch.empty(B.owq_backward_workspace_bytes(lin.handle, tokens), dtype=torch.uint8, device="cuda")
    B.owq_linear_backward(lin.handle, dyt.data_ptr(), xt.data_ptr(), guard.data_ptr(), 0, tokens, ws.data_ptr(), ws.numel())
    torch.cuda.synchronize()
    want, _ = backward.owq_backward_ref(layer.codes, layer.scale, layer.zero, group, layer.weak_idx, layer.weak_w, x, dy)
    got = guard.cpu().numpy()
    rel, mx = owq_ref.parity_errors(got[:tokens], want)
    assert rel <= 1e-3 and mx <= 1e-2, (rel, mx)
    assert (got[tokens] == 7).all()
    lin.close()


@pytest.mark.parametrize("bits,group,rows", [(3, 128, 1000), (4, 0, 70), (4, 256, 4200)])
@pytest.mark.parametrize("zeros", ["integers", "any"])
def test_step_sizes_up_to_the_largest(env, bits, group, rows, zeros):
    # Whatever finite step size and zero point a row has, its weights times its gradients add to the others: rows of step
    # sizes from 2^-6 to 65504, zero points to 1200, gradients so that all rows weigh alike.
    torch, B = env
    layer = make_layer(LayerSpec("bwdl", 900, rows, bits, group, 6, 7))
    rng = np.random.default_rng(12)
    s = np.exp2(rng.uniform(-6, 16, (rows, 1))) * np.ones(layer.scale.shape)
    layer.scale[:] = np.minimum(s * rng.choice([-1, 1], s.shape), 65504).astype(np.float16)
    layer.zero[rng.random(rows) < 0.2] = 1024
    if zeros == "any":
        layer.zero[:] = (layer.zero.astype(np.float32) + rng.normal(0, 2, layer.zero.shape)).astype(np.float16)
        layer.zero[rng.random(rows) < 0.05] = -1199
    layer.weak_w[:] = 0
    x = make_x(layer, 140)
    dy = (rng.normal(0, 0.05, (140, rows)) / np.abs(s[:, 0])).astype(np.float16)
    print(f"{rows} rows, groups of {group}, zero points: {zeros}", flush=True)
    lin = B.OwqLinear(layer, layout=1)
    dx, _ = lin.backward(torch.from_numpy(dy).cuda(), torch.from_numpy(x).cuda())
    lin.close()
    want, _ = backward.owq_backward_ref(layer.codes, layer.scale, layer.zero, group, layer.weak_idx, layer.weak_w, x, dy)
    keep = np.ones(900, bool)
    keep[layer.weak_idx] = False
    rel, mx = owq_ref.parity_errors(dx.cpu().numpy()[:, keep], want[:, keep])
    assert rel <= 1e-3 and mx <= 1e-2, (rel, mx)
