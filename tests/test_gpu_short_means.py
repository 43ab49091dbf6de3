"""Means of messages that one workgroup adds up by itself (at most 8,192 values), at the edges of its loop and of the rule, against
the exactly rounded mean of the oracle: equal bits."""
import numpy as np
import pytest

from rgc_testutil import GpuLayers

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rgc():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1808_04357_amd as pkg
    pkg.load_library()
    return pkg


@pytest.mark.parametrize("law", ["normal", "cancelling", "subnormal"])
@pytest.mark.parametrize("longest", [1, 255, 2048, 2049, 8191, 8192, 8193])
def test_means_around_the_length_one_workgroup_takes(rgc, oracle, longest, law):
    import torch
    g = np.random.default_rng(longest)
    sizes = [longest, max(1, longest - 1), (longest + 1) // 2, 1]
    V = []
    for n in sizes:
        v = g.standard_normal(n).astype(np.float32)
        if law == "cancelling":
            h = (v[:n // 2] * np.exp2(g.integers(-60, 90, n // 2))).astype(np.float32)
            v = np.concatenate([h, -h, np.full(n - 2 * (n // 2), 1e-30, np.float32)])
            g.shuffle(v)
        elif law == "subnormal":
            v = (g.integers(-2 ** 20, 2 ** 20, n).astype(np.float64) * 2.0 ** -149).astype(np.float32)
        V.append(v)
    dev = GpuLayers(rgc, [np.zeros(n, np.float32) for n in sizes], sizes)
    for l in range(len(sizes)):
        dev.out_val[l].copy_(torch.from_numpy(V[l]))
    counts = sizes[:-1] + [0]                                    # a message of no values: mean 0
    dev.out_count.copy_(torch.tensor(counts, dtype=torch.int32))
    ctx = rgc.Context(sum(sizes), len(sizes))
    means = torch.full((len(sizes),), 7.0, dtype=torch.float32, device=torch.device("cuda:0"))
    print("  means: longest %d, %s" % (longest, law), flush=True)
    rgc.rgc_message_means(ctx, dev.layers, means, torch.cuda.current_stream())
    got = means.cpu().numpy()
    ctx.close()
    assert got[-1].view(np.uint32) == 0
    for l, n in enumerate(counts[:-1]):
        _, want, c = oracle.compress_layer_asq(np.zeros(n, np.float32), V[l].copy(), n, +1)
        assert c == n
        assert got[l].view(np.uint32) == np.float32(want).view(np.uint32), (l, n, got[l], want)
