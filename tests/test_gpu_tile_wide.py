"""GPU parity of the kernels for more than 64 tokens (tile layout) against the fp64 CPU oracle: the edges of their
256-row x 64-token tiles and 128-column blocks, rows off the 16-byte grid, one and several chunks of 128 weak
columns, zero points that are no small integers, split and unsplit columns.

Bar: relative L2 error <= 1e-3 and max-abs error <= 1e-2 * rms(y) over the output and per token, as for the other
kernels of the layout (what is rounded is y, to fp16: 2^-11 / sqrt(3) = 2.8e-4)."""
import zlib

import numpy as np
import pytest

from oracle import owq_ref
from synth import LayerSpec, make_layer, make_x

pytestmark = pytest.mark.gpu

REL_L2, MAX_ABS, TILE = 1e-3, 1e-2, 1


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
        assert rel <= REL_L2 and mx <= MAX_ABS, (what, rel, mx)


CASES = [
    # name, d_in, d_out, bits, group, k, tokens
    ("w3_first", 512, 256, 3, 128, 8, 65),
    ("w4_tile", 512, 256, 4, 128, 8, 128),
    ("w3_tile1", 640, 257, 3, 128, 8, 129),          # odd number of blocks, one row in the second row group
    ("w4_ch_split", 2048, 70, 4, 0, 20, 192),        # few tiles: columns are split
    ("w3_ch", 256, 600, 3, 0, 24, 100),              # one pair of blocks: no split
    ("w3_g256", 1536, 40, 3, 256, 5, 70),
    ("w4_ragged", 1001, 333, 4, 128, 7, 99),         # rows of x are no multiple of 16 bytes
    ("w3_ragged8", 1000, 48, 3, 0, 7, 77),           # they are, but not of a block
    ("w4_one_block", 100, 33, 4, 0, 3, 66),
    ("w3_two_chunks", 1024, 64, 3, 128, 200, 80),    # weak columns: a whole chunk of 128 and a part of one
    ("w4_all_weak", 128, 40, 4, 0, 128, 67),
    ("w3_k0", 768, 64, 3, 128, 0, 90),
    ("w4_rounds", 256, 4096, 4, 128, 4, 2100),       # more tiles than run at once
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("zeros", ["integers", "any"])
def test_layers_match_oracle(env, case, zeros):
    torch, B = env
    name, d_in, d_out, bits, group, k, tokens = case
    layer = make_layer(LayerSpec(name, d_in, d_out, bits, group, k, zlib.crc32(name.encode()) % 10000))
    if zeros == "any":       # fractions, and values whose difference to a code is no fp16 number
        rng = np.random.default_rng(5)
        z = layer.zero.astype(np.float32) + rng.normal(0, 2, layer.zero.shape)
        z[rng.random(z.shape) < 0.05] = 1500.5
        z[rng.random(z.shape) < 0.05] = -3000.0
        layer.zero[:] = z.astype(np.float16)
    x = make_x(layer, tokens)
    print(f"case {name}, zero points: {zeros}", flush=True)
    lin = B.OwqLinear(layer, layout=TILE)
    y = lin(torch.from_numpy(x).cuda()).cpu().numpy()
    want = owq_ref.owq_linear_layer(layer, x)
    check(y, want, name)
    # the passes of at most 64 tokens give the same layer, to the rounding of y
    part = np.concatenate([lin(torch.from_numpy(x[i:i + 64].copy()).cuda()).cpu().numpy() for i in range(0, tokens, 64)])
    check(part, want, name + " in passes")
    lin.close()


def test_rows_and_results_off_the_grid(env):
    torch, B = env
    layer = make_layer(LayerSpec("off", 512, 264, 3, 128, 16, 61))
    x = make_x(layer, 70)
    want = owq_ref.owq_linear_layer(layer, x)
    lin = B.OwqLinear(layer, layout=TILE)
    xb = torch.zeros(70 * 512 + 8, dtype=torch.float16, device="cuda")
    yb = torch.full((70 * 264 + 16,), 7.0, dtype=torch.float16, device="cuda")
    for xo, yo in ((1, 1), (0, 3), (5, 0)):
        print(f"x off by {xo}, y off by {yo} elements", flush=True)
        xb[xo:xo + 70 * 512] = torch.from_numpy(x).cuda().flatten()
        yb.fill_(7.0)
        B.owq_linear(lin.handle, xb.data_ptr() + 2 * xo, yb.data_ptr() + 2 * yo, 70)
        got = yb.cpu().numpy()
        check(got[yo:yo + 70 * 264].reshape(70, 264), want, (xo, yo))
        assert (got[:yo] == 7.0).all() and (got[yo + 70 * 264:] == 7.0).all()
    lin.close()


def test_weak_positions_do_not_leak_and_runs_agree(env):
    torch, B = env
    layer = make_layer(LayerSpec("leakw", 1000, 300, 4, 128, 9, 62))
    layer.weak_w[:] = 0
    x = make_x(layer, 130)
    x2 = x.copy()
    x2[:, layer.weak_idx] = np.float16(30000.0)
    x2[77, layer.weak_idx[0]] = np.float16(np.inf)
    lin = B.OwqLinear(layer, layout=TILE)
    a = lin(torch.from_numpy(x).cuda()).cpu().numpy()
    b = lin(torch.from_numpy(x2).cuda()).cpu().numpy()
    keep = np.arange(130) != 77           # 0 * inf in that token's weak product
    np.testing.assert_array_equal(a[keep].view(np.uint16), b[keep].view(np.uint16))
    np.testing.assert_array_equal(a.view(np.uint16), lin(torch.from_numpy(x).cuda()).cpu().numpy().view(np.uint16))
    lin.close()


def test_integer_inputs_are_bit_exact(env):
    """Integer activations and zero points, step size 1, no weak columns: every sum is an integer below 2^24."""
    torch, B = env
    layer = make_layer(LayerSpec("intw", 768, 300, 3, 128, 0, 63))
    layer.scale[:] = np.float16(1.0)
    x = np.random.default_rng(6).integers(-8, 9, (150, 768)).astype(np.float16)
    lin = B.OwqLinear(layer, layout=TILE)
    y = lin(torch.from_numpy(x).cuda()).cpu().numpy()
    np.testing.assert_array_equal(y, owq_ref.owq_linear_layer(layer, x).astype(np.float16))
    lin.close()
