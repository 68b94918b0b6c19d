"""Several sets of weak columns on the tile layout: more than one chunk of 128 weak columns (a last one that is whole, ragged,
of one unit), passes of 32 tokens or fewer and of more, rows that are no multiple of 64, tokens that use no set, one set or
all of them.  Bar as in test_gpu_multi: relative L2 error <= 1e-3, max-abs <= 1e-2 rms, per token."""
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


@pytest.mark.parametrize("k", [130, 200, 256, 300])
@pytest.mark.parametrize("batch", [3, 17, 32, 33, 64, 100])
@pytest.mark.parametrize("use", ["none", "one", "all"])
def test_chunks_of_weak_columns(env, k, batch, use):
    torch, B = env
    d_in, d_out, n_sets = 900, 170 if batch % 2 else 333, 6
    bits, group = (3, 0) if k in (130, 256) else (4, 128)
    layer = make_layer(LayerSpec("chunks", d_in, d_out, bits, group, k, k + batch))
    rng = np.random.default_rng(k * batch)
    sets = [rng.normal(0, 0.02, size=(d_out, k)).astype(np.float16) for _ in range(n_sets)]
    if use == "none":
        task = np.full(batch, -1, dtype=np.int32)
    elif use == "one":
        task = np.where(rng.random(batch) < 0.5, 4, n_sets).astype(np.int32)         # n_sets: the layer's own
    else:
        task = ((np.arange(batch) + rng.integers(0, 2, batch)) % (n_sets + 1) - 1).astype(np.int32)
    x = make_x(layer, batch)
    print(f"k {k}, batch {batch}, sets: {use}", flush=True)
    lin = B.OwqLinear(layer, layout=1)
    table, bufs = lin.add_weak_sets(sets)
    y = lin.multi(torch.from_numpy(x).cuda(), table, torch.from_numpy(task).cuda()).cpu().numpy()
    want = owq_ref.owq_linear_multi_ref(layer.codes, layer.scale, layer.zero, layer.group_size, layer.weak_idx, sets + [layer.weak_w],
                                        [t if 0 <= t < n_sets else n_sets for t in task], x)
    for n in range(batch):
        rel, mx = owq_ref.parity_errors(y[n], want[n])
        assert rel <= 1e-3 and mx <= 1e-2, (n, task[n], rel, mx)
    lin.close()


@pytest.mark.parametrize("d_out,batch", [(10240, 64), (10250, 33), (10250, 64), (24576, 32), (24600, 5), (24600, 32), (24600, 40)])
@pytest.mark.parametrize("bits,group,k,used", [(3, 0, 130, 6), (4, 128, 20, 1)])
def test_many_rows(env, d_out, batch, bits, group, k, used):
    # either side of the rows from which a workgroup of the last launch takes 64 of them: by the number of tokens
    torch, B = env
    n_sets = 6
    layer = make_layer(LayerSpec("rows", 256, d_out, bits, group, k, d_out + batch))
    rng = np.random.default_rng(d_out + batch)
    sets = [rng.normal(0, 0.02, size=(d_out, k)).astype(np.float16) for _ in range(n_sets)]
    task = (rng.integers(-1, n_sets, batch) if used > 1 else np.full(batch, 2)).astype(np.int32)
    x = make_x(layer, batch)
    print(f"{d_out} rows, {batch} tokens, k {k}", flush=True)
    lin = B.OwqLinear(layer, layout=1)
    table, bufs = lin.add_weak_sets(sets)
    y = lin.multi(torch.from_numpy(x).cuda(), table, torch.from_numpy(task).cuda()).cpu().numpy()
    want = owq_ref.owq_linear_multi_ref(layer.codes, layer.scale, layer.zero, layer.group_size, layer.weak_idx, sets + [layer.weak_w],
                                        [t if 0 <= t < n_sets else n_sets for t in task], x)
    for n in range(batch):
        rel, mx = owq_ref.parity_errors(y[n], want[n])
        assert rel <= 1e-3 and mx <= 1e-2, (n, task[n], rel, mx)
    lin.close()


@pytest.mark.parametrize("d_out,k", [(40, 1), (200, 30), (96, 33), (170, 64), (128, 130), (300, 200), (70, 300), (10300, 70)])
@pytest.mark.parametrize("bits,group", [(3, 0), (4, 128)])
@pytest.mark.parametrize("batch", [33, 64])
def test_one_task_equals_the_plain_call_bit_for_bit(env, d_out, k, bits, group, batch):
    # 33 to 64 tokens, the plain call's three launches: sums of more than two k-steps in the same order, beside tokens of other tasks too
    torch, B = env
    layer = make_layer(LayerSpec("same", 900, d_out, bits, group, k, d_out + k))
    x = torch.from_numpy(make_x(layer, batch)).cuda()
    rng = np.random.default_rng(k)
    sets = [layer.weak_w] + [rng.normal(0, 0.02, size=(d_out, k)).astype(np.float16) for _ in range(5)]
    print(f"{d_out} rows, {batch} tokens, k {k}", flush=True)
    lin = B.OwqLinear(layer, layout=1)
    table, bufs = lin.add_weak_sets(sets)
    want = lin(x).cpu().numpy().view(np.uint16)
    for task in (np.zeros(batch), np.full(batch, -1), np.where(rng.random(batch) < 0.4, 0, rng.integers(1, 6, batch))):
        y = lin.multi(x, table, torch.from_numpy(task.astype(np.int32)).cuda()).cpu().numpy().view(np.uint16)
        np.testing.assert_array_equal(y[task <= 0], want[task <= 0])
    lin.close()
