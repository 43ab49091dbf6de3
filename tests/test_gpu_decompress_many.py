"""GPU parity of the decompression around the largest numbers of workers its tile kernels take (bit equality)."""
import numpy as np
import pytest

from test_gpu_decompress import compare, gpu_decompress, oracle_all, random_messages

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rgc():
    import paper_1808_04357_amd as m
    return m


@pytest.mark.parametrize("add", [False, True])
@pytest.mark.parametrize("workers", [127, 129, 255, 256, 257])
def test_around_the_limits(rgc, oracle, workers, add):
    """Few and many entries per tile, hot positions hit by nearly every worker, more of them in one tile than it has
    rows, messages that run beyond a worker's window, empty ones, tiles that end with the layer."""
    g = np.random.default_rng(workers)
    sizes = [3 * 8192 + 77, 8192, 511, 40_003]
    hot = [g.choice(n, size=min(n, 200), replace=False) for n in sizes]
    idx, val = random_messages(g, sizes, workers, [60, 300, 20, 12], hot=hot)
    for w in range(0, workers, 7):
        idx[w][0], val[w][0] = idx[w][0][:0], val[w][0][:0]
    for w in (1, workers - 1):                                  # far beyond the window
        idx[w][1] = np.arange(0, 8192, 3, dtype=np.int32)
        val[w][1] = g.standard_normal(idx[w][1].size).astype(np.float32)
    init = [g.standard_normal(n).astype(np.float32) for n in sizes] if add else None
    ctx = rgc.Context(sum(sizes), len(sizes))
    got = gpu_decompress(rgc, ctx, idx, val, sizes, 1.0 / workers, init, misalign=workers % 2)
    compare("%d workers" % workers, got, oracle_all(oracle, idx, val, sizes, 1.0 / workers, init))
    ctx.close()


def test_a_changed_list_is_checked_again(rgc):
    """A message list that differs in one field from the one of the call before is looked through like a new one."""
    import torch
    ctx = rgc.Context(1000, 1)
    idx = [[torch.arange(8, dtype=torch.int32, device="cuda")] for _ in range(40)]
    val = [[torch.ones(8, device="cuda")] for _ in range(40)]
    dense = [torch.empty(1000, device="cuda")]
    msgs = rgc.MessageList(idx, val, dense)
    for _ in range(2):
        rgc.rgc_decompress_accumulate(ctx, msgs, 1.0)
    torch.cuda.synchronize()
    assert float(dense[0][7]) == 40.0 and float(dense[0][8]) == 0.0
    for w, field, bad in ((3, "count", 1001), (17, "count", -1), (39, "val", None), (38, "idx", msgs.msgs[38].idx + 2)):
        keep = getattr(msgs.msgs[w], field)
        setattr(msgs.msgs[w], field, bad)
        with pytest.raises(rgc.RgcError):
            rgc.rgc_decompress_accumulate(ctx, msgs, 1.0)
        setattr(msgs.msgs[w], field, keep)
    msgs.msgs[5].count = 4
    rgc.rgc_decompress_accumulate(ctx, msgs, 1.0)
    torch.cuda.synchronize()
    assert float(dense[0][3]) == 40.0 and float(dense[0][7]) == 39.0
    ctx.close()
