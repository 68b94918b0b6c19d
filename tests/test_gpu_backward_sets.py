"""Backward where the work of one set of launches is cut: every remainder of a range's last step of four row tiles, in
either half of the range; staging blocks of one and of four token tiles; five and more passes of 128 tokens at once, and
batches that still need several sets.  Bar as in test_gpu_backward: relative L2 error <= 1e-3, max-abs <= 1e-2 rms."""
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
    # ranges of 1 to 9 row tiles (16 ranges at most)
    (256, 16 * 32, 3, 0, 4, 20), (256, 33 * 32, 4, 128, 4, 20), (256, 47 * 32, 3, 128, 4, 20), (256, 64 * 32 - 7, 4, 0, 4, 20),
    (200, 80 * 32, 3, 128, 4, 20), (256, 95 * 32, 4, 128, 4, 20), (256, 110 * 32 + 1, 3, 0, 4, 20), (256, 128 * 32, 4, 128, 4, 20),
    (256, 141 * 32, 3, 128, 4, 20),
    (512, 96, 4, 128, 5, 700), (300, 200, 3, 0, 9, 2300),          # six passes in one set; nine, twice
    (128, 33000, 4, 0, 3, 140), (128, 66000, 3, 0, 2, 800),        # staging blocks of four token tiles; sets of four passes
])
def test_cuts(env, d_in, d_out, bits, group, k, tokens):
    torch, B = env
    layer = make_layer(LayerSpec("sets", d_in, d_out, bits, group, k, d_in + d_out))
    rng = np.random.default_rng(d_out)
    x = make_x(layer, tokens)
    dy = rng.normal(0, 0.05, (tokens, d_out)).astype(np.float16)
    print(f"{d_in} -> {d_out}, {bits} bit, group {group}, {tokens} tokens", flush=True)
    lin = B.OwqLinear(layer, layout=1)
    dx, dww = lin.backward(torch.from_numpy(dy).cuda(), torch.from_numpy(x).cuda())
    want_dx, want_dww = backward.owq_backward_ref(layer.codes, layer.scale, layer.zero, group, layer.weak_idx, layer.weak_w, x, dy)
    rel, mx = owq_ref.parity_errors(dx.cpu().numpy(), want_dx)
    assert rel <= 1e-3 and mx <= 1e-2, (rel, mx)
    rel, _ = owq_ref.parity_errors(dww.cpu().numpy(), want_dww)
    assert rel <= 1e-5, rel
    again, _ = lin.backward(torch.from_numpy(dy).cuda(), torch.from_numpy(x).cuda())
    np.testing.assert_array_equal(dx.cpu().numpy().view(np.uint16), again.cpu().numpy().view(np.uint16))
    lin.close()


@pytest.mark.parametrize("d_in,d_out", [(4096, 4096), (1664, 768), (5120, 5120), (2048, 2048), (768, 7040), (16384, 512), (1024, 30000)])
def test_a_workspace_serves_smaller_batches(env, d_in, d_out):
    # from four passes of 128 tokens on, as a caller that asks once for its largest batch has it
    torch, B = env
    desc = B.make_desc(d_out, d_in, 4, 128, d_in // 100, layout=1)
    buf = torch.empty(B.owq_packed_bytes(desc), dtype=torch.uint8, device="cuda")
    handle = B.owq_open_packed(desc, buf.data_ptr(), buf.numel())
    sizes = [B.owq_backward_workspace_bytes(handle, b) for b in range(385, 2600, 43)]
    B.owq_free_layer(handle)
    assert sizes == sorted(sizes)


@pytest.mark.parametrize("d_in,d_out", [(16384, 4096), (13824, 5120), (11008, 4096), (4096, 16384), (640, 200)])
def test_a_workspace_serves_every_smaller_batch(env, d_in, d_out):
    # also those of fewer than four passes, where rows are cut into ranges that a larger batch does without
    torch, B = env
    desc = B.make_desc(d_out, d_in, 4, 128, d_in // 100, layout=1)
    buf = torch.empty(B.owq_packed_bytes(desc), dtype=torch.uint8, device="cuda")
    handle = B.owq_open_packed(desc, buf.data_ptr(), buf.numel())
    sizes = [B.owq_backward_workspace_bytes(handle, b) for b in list(range(1, 1200, 31)) + [2048, 4096]]
    B.owq_free_layer(handle)
    assert sizes == sorted(sizes)
