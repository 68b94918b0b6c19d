"""The last of the batched path's three launches where one task's weak columns are dealt out to its waves: no weak columns, one
k-step, parts of a chunk of 128 and more than two of them; rows that are no multiple of 32; 32 tokens or fewer and more; and
either side of the numbers of rows from which a workgroup takes 64 of them (more than 32 tokens; fewer).  Bar as for the other kernels of the layout."""
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


@pytest.mark.parametrize("d_in,d_out,k", [(900, 33, 0), (900, 170, 5), (520, 65, 100), (900, 300, 130), (900, 95, 300),
                                          (256, 10240, 9), (256, 10250, 9), (256, 24576, 9), (256, 24600, 9)])
@pytest.mark.parametrize("bits,group", [(3, 0), (4, 128)])
@pytest.mark.parametrize("batch", [1, 32, 33, 64])
def test_weak_columns_dealt_out_to_the_waves(env, d_in, d_out, k, bits, group, batch):
    torch, B = env
    layer = make_layer(LayerSpec("finish", d_in, d_out, bits, group, k, d_out + k))
    x = make_x(layer, batch)
    print(f"{d_in} -> {d_out}, k {k}, {bits} bit, group {group}, {batch} tokens", flush=True)
    lin = B.OwqLinear(layer, layout=1)
    B.owq_set_launch(lin.handle, prefetch_depth=-1)          # three launches, whatever the number of tokens
    y = lin(torch.from_numpy(x).cuda()).cpu().numpy()
    want = owq_ref.owq_linear_layer(layer, x)
    for n in range(batch):
        rel, mx = owq_ref.parity_errors(y[n], want[n])
        assert rel <= 1e-3 and mx <= 1e-2, (n, rel, mx)
    lin.close()
