"""GPU parity of small calls at high densities: edges of their wave-chunks, of the groups that elect a layer's last workgroup, and
of the members that one workgroup's LDS holds (bit equality)."""
import numpy as np
import pytest

from rgc_testutil import GpuLayers, assert_layers_equal, oracle_step

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rgc():
    import paper_1808_04357_amd as m
    return m


@pytest.mark.parametrize("momentum", [False, True])
@pytest.mark.parametrize("ppm", [62_500, 250_000])
@pytest.mark.parametrize("sizes", [[2047, 2048, 2049, 4 * 2048, 4 * 2048 + 1, 300_001], [32 * 4 * 2048, 32 * 4 * 2048 + 1, 64 * 2048 - 3], [700_001]])
def test_chunk_edges(rgc, oracle, sizes, ppm, momentum):
    """Wave-chunks of 2048 elements, workgroups of four of them, groups of 32 workgroups: one element less, none, one more."""
    g = np.random.default_rng(ppm + sizes[0])
    ks = [rgc.rgc_k_for_density(n, ppm) for n in sizes]
    V = [(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes]
    U = [(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] if momentum else None
    dev = GpuLayers(rgc, V, ks, U, misalign=1)
    ctx = rgc.Context(sum(sizes), len(sizes))
    large = [l for l, n in enumerate(sizes) if n > 1 << 15]             # (smaller layers need no list)
    assert large
    ranked = 0
    for t in range(6):
        G = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
        dev.set_grads(G)
        dev.step(ctx, 0.3 if momentum else 0.0)
        msgs = oracle_step(oracle, G, V, ks, U, m=0.3 if momentum else 0.0)
        assert_layers_equal("step %d" % t, ks, dev.results(), msgs, V, U)
        stats = ctx.last_stats(len(sizes))
        ranked += all(stats[l][0] == 0 and stats[l][2] > 0 for l in large)
    assert ranked >= 2                                                  # calls whose large layers were ranked from their lists
    ctx.last_error()
    ctx.close()


@pytest.mark.parametrize("more", [0, 1])
def test_largest_call_on_short_chunks(rgc, oracle, more):
    """Calls of 2^21 elements take wave-chunks of 2048 elements, of one more 4096: values anywhere, and in one stretch of twenty."""
    g = np.random.default_rng(more)
    sizes = [1_900_001, (1 << 21) - 1_900_001 + more]
    ks = [rgc.rgc_k_for_density(n, 62_500) for n in sizes]
    V = [np.zeros(n, np.float32) for n in sizes]
    dev = GpuLayers(rgc, V, ks)
    ctx = rgc.Context(sum(sizes), len(sizes))
    ranked = 0
    for t in range(8):
        G = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
        if t >= 4:
            G = [x * (g.random(-(-x.size // 2048)) < 0.05).repeat(2048)[:x.size] for x in G]
        dev.set_grads(G)
        dev.step(ctx)
        msgs = oracle_step(oracle, G, V, ks)
        assert_layers_equal("step %d" % t, ks, dev.results(), msgs, V)
        ranked += sum(s[0] == 0 and s[2] > 0 for s in ctx.last_stats(len(sizes)))
    assert ranked >= 2
    ctx.last_error()
    ctx.close()


@pytest.mark.parametrize("ties", [1500, 2040, 2060, 3000])
def test_members_in_lds_and_not(rgc, oracle, ties):
    """The k-th key is shared by `ties` elements on every call, and up to 2048 members are ranked in LDS."""
    g = np.random.default_rng(ties)
    n, k = 1_200_000, 75_000
    order = g.permutation(n)
    large, tied, rest = order[:k - ties // 2], order[k - ties // 2:k + ties - ties // 2], order[k + ties - ties // 2:]
    v = np.zeros(n, np.float32)
    v[rest] = g.uniform(0.0, 0.9, rest.size).astype(np.float32)
    V = [v]
    dev = GpuLayers(rgc, V, [k])
    ctx = rgc.Context(n, 1)
    for t in range(5):
        grad = np.zeros(n, np.float32)
        grad[large] = g.uniform(1.5, 4.0, large.size).astype(np.float32)
        grad[tied] = 1.0 - V[0][tied]                 # what is left of them is 1 or 0: exact
        dev.set_grads([grad])
        dev.step(ctx)
        msgs = oracle_step(oracle, [grad], V, [k])
        assert_layers_equal("step %d" % t, [k], dev.results(), msgs, V)
    assert ctx.last_paths(1) == [0]
    assert ctx.last_stats(1)[0][2] >= ties
    ctx.last_error()
    ctx.close()
