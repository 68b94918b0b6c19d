"""Which kernels prompts go to: workgroups of eight waves (512 threads) or of four, read from a captured call.  The figures are
those of the plan's comments: calls that eight waves make slower stay with four, and calls that they make faster get them."""
import types

import numpy as np
import pytest

from launches import launches

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


@pytest.mark.parametrize("d_in,d_out,bits,group,tokens,eight", [
    (3968, 7345, 4, 0, 1352, False),       # one scale per row: tiles of 64 tokens are a whole round
    (6400, 8456, 4, 0, 1978, False),       # ... two launches, of which eight waves would be one
    (10240, 10871, 3, 0, 1390, False),     # ... two rounds of eight waves, nothing cut
    (8192, 5120, 3, 0, 2040, True),        # ... one launch, cut
    (11264, 6137, 4, 256, 1327, False),    # groups: 8 tiles would be cut into 22 ranges each
    (9600, 4752, 3, 256, 1690, True),      # ... 10 tiles into 19, two launches otherwise
    (9856, 3808, 3, 128, 1563, True),      # ... one round, nothing cut
    (5120, 13824, 4, 128, 1500, False)])   # 648 tiles: two workgroups of four waves on every compute unit
def test_waves_of_a_prompt(env, d_in, d_out, bits, group, tokens, eight):
    torch, B = env
    groups = -(-d_in // group) if group else 1
    one = np.ones((d_out, groups), dtype=np.float16)
    layer = types.SimpleNamespace(d_out=d_out, d_in=d_in, bits=bits, group_size=group, k=1, codes=np.zeros((d_out, d_in), dtype=np.uint8),
                                  scale=one, zero=one, weak_idx=np.array([3], dtype=np.int32), weak_w=np.zeros((d_out, 1), dtype=np.float16))
    lin = B.OwqLinear(layer, layout=1)
    x = torch.zeros((tokens, d_in), dtype=torch.float16, device="cuda")
    y = torch.empty((tokens, d_out), dtype=torch.float16, device="cuda")
    got = launches(torch, lambda: lin(x, out=y))
    print(f"{d_in} -> {d_out}, {tokens} tokens: {got}", flush=True)
    assert any(threads == 512 for _, threads in got) == eight
    lin.close()
