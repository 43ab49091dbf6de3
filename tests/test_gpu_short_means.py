"""The ends of exactly rounded sums.  Means of messages that one workgroup adds up by itself (at most 8,192 values), at the edges of its loop and of the rule, against
the exactly rounded mean of the oracle: equal bits; and sums whose rounding
hangs on a term far below the last bit."""
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


@pytest.mark.parametrize("tiny", [2.0 ** -120, 0.0, -2.0 ** -120])
def test_rounding_decided_by_the_smallest_term(rgc, oracle, tiny):
    """Sum = 1 + 2^-24 + 2^-53 + tiny: half way between two doubles but for `tiny`, and the lower one half way between two
    floats.  The pieces lie in parts of 2,048 values of their own, so that the smallest reaches the final rounding as the
    error of an error."""
    import torch
    n = 16_384
    v = np.zeros(n, np.float32)
    v[[0, 1, 2]] = [1.0, 2.0 ** -24, 2.0 ** -54]
    v[2_048] = 2.0 ** -54
    v[[4_096, 4_097]] = [2.0 ** -40, tiny]
    v[6_144] = -2.0 ** -40
    dev = GpuLayers(rgc, [np.zeros(n, np.float32)], [n])
    dev.out_val[0].copy_(torch.from_numpy(v))
    dev.out_count.copy_(torch.tensor([n], dtype=torch.int32))
    ctx = rgc.Context(n, 1)
    means = torch.full((1,), 7.0, dtype=torch.float32, device=torch.device("cuda:0"))
    print("  rounding: tiny %r" % tiny, flush=True)
    rgc.rgc_message_means(ctx, dev.layers, means, torch.cuda.current_stream())
    got = means.cpu().numpy()[0]
    ctx.close()
    want = np.float32((1.0 + 2.0 ** -23 if tiny > 0.0 else 1.0) / n)
    _, omean, _ = oracle.compress_layer_asq(np.zeros(n, np.float32), v.copy(), n, +1)
    assert want == np.float32(omean)
    assert got.view(np.uint32) == want.view(np.uint32)
