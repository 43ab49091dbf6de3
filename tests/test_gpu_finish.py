"""GPU parity of the tiled calls (bit equality): layers selected from the residual itself (up to 32768 elements), layers
ended by one workgroup from their candidate lists, larger layers in parts of 2^20 elements, and the launch that takes the
layers whose hint missed."""
import numpy as np
import pytest

from rgc_testutil import GpuLayers, assert_layers_equal, oracle_step, u32
from test_gpu_compress import run_iterations

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rgc():
    import paper_1808_04357_amd as m
    return m


DIRECT = [1, 2, 3, 4, 5, 63, 64, 65, 1023, 1024, 1025, 4095, 4097, 16385, 32767, 32768]


@pytest.mark.parametrize("law", ["normal", "ties", "sparse", "constant", "special"])
@pytest.mark.parametrize("share", ["one", "permille", "quarter", "all"])
def test_direct_layers(rgc, oracle, law, share):
    g = np.random.default_rng(5)

    def draw(n, s):
        a = (g.standard_normal(n) * s).astype(np.float32)
        if law == "ties":
            a = (np.round(a / s * 3) / 3).astype(np.float32)
        elif law == "sparse":
            a[g.random(n) < 0.95] = 0.0
        elif law == "constant":
            a[:] = -1.5
        elif law == "special" and n > 3:
            a[g.integers(0, n, 3)] = [np.nan, np.inf, -np.inf]
            a[: n // 3] = g.integers(-5, 5, n // 3) * np.float32(1.4e-45)
        return a

    ks = [{"one": 1, "permille": rgc.rgc_k_for_density(n), "quarter": max(1, n // 4), "all": n}[share] for n in DIRECT]
    V = [draw(n, 1.0) for n in DIRECT]
    G_list = [[draw(n, 0.25) if law != "constant" else np.zeros(n, np.float32) for n in DIRECT] for _ in range(2)]
    run_iterations(rgc, oracle, V, G_list, ks, misalign=1, tag="direct %s %s" % (law, share))


def test_direct_layers_with_momentum_and_without_hints(rgc, oracle):
    g = np.random.default_rng(6)
    V = [(g.standard_normal(n)).astype(np.float32) for n in DIRECT]
    U = [(g.standard_normal(n)).astype(np.float32) for n in DIRECT]
    G_list = [[(g.standard_normal(n)).astype(np.float32) for n in DIRECT] for _ in range(3)]
    ks = [max(1, n // 50) for n in DIRECT]
    for flags in (0, rgc.RGC_NESTEROV, rgc.RGC_NO_MOMENTUM_MASK | rgc.RGC_NO_HINTS):
        run_iterations(rgc, oracle, V, G_list, ks, U0=U, m=0.9, flags=flags, tag="direct momentum %x" % flags)


# 32769 is the smallest layer taken from its lists; 2457 entries sent (rank 6142 aimed at) and 1024 tiles of 4096 elements the
# most one workgroup takes
@pytest.mark.parametrize("sizes,ks", [([32769, 32768, 100], None), ([65536 + 1023, 40_000], None), ([1 << 20], None),
                                      ([2_457_000, 1_000_003, 33_000], None), ([400_000], [2457]), ([400_000], [2458]),
                                      ([3 << 20], None), ([(3 << 20) - 1, 5 << 20, 70_000], None), ([(3 << 20) + 1], None),
                                      ([1024 * 4096], [400]), ([1024 * 4096 + 1], [400]),
                                      ([700_000, 500_000, 300], [1, 2, 3])])
def test_layers_from_their_lists(rgc, oracle, sizes, ks):
    g = np.random.default_rng(7)
    ks = ks or [rgc.rgc_k_for_density(n) for n in sizes]
    V = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
    U = [(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes]
    G_list = [[(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] for _ in range(5)]
    paths = run_iterations(rgc, oracle, V, G_list, ks, U0=U, m=0.9, threads=8, tag="lists")
    assert any(p[0] == 0 for p in paths[1:]), paths


def test_long_lists_of_a_layer_ended_by_one_workgroup(rgc, oracle):
    """The large values sit in 275 of 733 tiles, more than the 16 in each that are asked for with the list's length, and one
    tile has far more of them than the others."""
    g = np.random.default_rng(8)
    n, k = 3_000_000, 2457
    scale = np.full(n, 1e-3, np.float32)
    scale[: 1100 * 1024] = 1.0
    scale[5 * 1024:6 * 1024] = 1.6
    V = [(g.standard_normal(n).astype(np.float32) * scale)]
    G_list = [[(g.standard_normal(n).astype(np.float32) * scale * 0.2)] for _ in range(4)]
    paths = run_iterations(rgc, oracle, V, G_list, [k], threads=8, tag="queue")
    assert any(p == [0] for p in paths[1:]), paths


@pytest.mark.parametrize("sizes", [[32768, 5000, 1], [200_000, 32768, 300]])
def test_reported_paths_of_small_layers(rgc, oracle, sizes):
    """A layer small enough to need no hint is on the one-pass path like the others: from the first call that has hints on."""
    g = np.random.default_rng(14)
    ks = [rgc.rgc_k_for_density(n) for n in sizes]
    V = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
    G_list = [[(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] for _ in range(4)]
    paths = run_iterations(rgc, oracle, V, G_list, ks, tag="paths")
    assert paths[0] == [1] * len(sizes) and all(p[-1] == 0 and p[-2] == 0 for p in paths[1:]), paths
    paths = run_iterations(rgc, oracle, V, G_list, ks, flags=rgc.RGC_NO_HINTS, tag="paths without hints")
    assert all(p == [1] * len(sizes) for p in paths), paths


# a full part (2^20 elements) has more than the 12288 candidates of one step from about 0.47 % on; 11,700 ppm is about the most that
# calls of more than 7 Mi elements count on a tile's list for
@pytest.mark.parametrize("ppm", [4000, 5000, 8000, 10_000, 11_500])
@pytest.mark.parametrize("momentum", [False, True])
def test_densities_up_to_one_percent_keep_their_hints(rgc, oracle, ppm, momentum):
    g = np.random.default_rng(12)
    sizes = [(2 << 20) + 77_777, 1 << 20, 600_000, 40_000, 3000]
    ks = [rgc.rgc_k_for_density(n, ppm) for n in sizes]
    V = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
    U = [(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] if momentum else None
    G_list = [[(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] for _ in range(8)]
    paths = run_iterations(rgc, oracle, V, G_list, ks, U0=U, m=0.9 if momentum else 0.0, threads=8, tag="%d ppm" % ppm)
    assert all(p[:4] == [0, 0, 0, 0] for p in paths[-4:]), paths


@pytest.mark.parametrize("ppm", [12_500, 15_625, 22_000])
@pytest.mark.parametrize("sizes", [[(1 << 20) + 77_777, 4096 * 40, 33_000, 300], [(7 << 20) - 40_000, 40_000], [(7 << 20) - 40_000, 40_001]])
def test_densities_up_to_two_percent_in_calls_of_up_to_seven_million_elements(rgc, oracle, ppm, sizes):
    """Tiled up to 7 Mi elements (the first two lists), dense layers above (the third), which have no hint where the optional
    scratch is not to be had; a tiled call needs none.  With it, both keep their hints."""
    g = np.random.default_rng(16)
    ks = [rgc.rgc_k_for_density(n, ppm) for n in sizes]
    V = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
    U = [(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes]
    G_list = [[(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] for _ in range(8)]
    tiled = sum(sizes) <= 7 << 20
    for limit in (0, -1):
        ctx = rgc.Context(sum(sizes), len(sizes))
        ctx.limit_optional_scratch(limit)
        paths = run_iterations(rgc, oracle, V, G_list, ks, U0=U, m=0.9, ctx=ctx, threads=8, tag="%d ppm, limit %d" % (ppm, limit))
        ctx.close()
        hinted = [l for l, n in enumerate(sizes) if n > 32768]
        want = 0 if tiled or limit < 0 else 1
        assert all(p[l] == want for p in paths[-3:] for l in hinted), paths


def test_most_that_large_calls_count_on_a_list_for(rgc, oracle):
    """More than 7 Mi elements at 11,500 ppm, with lists that need no optional scratch."""
    g = np.random.default_rng(20)
    sizes = [(7 << 20) - 5, 300_000, 60_001]
    ks = [rgc.rgc_k_for_density(n, 11_500) for n in sizes]
    V = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
    G_list = [[(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] for _ in range(6)]
    ctx = rgc.Context(sum(sizes), len(sizes))
    ctx.limit_optional_scratch(0)
    paths = run_iterations(rgc, oracle, V, G_list, ks, ctx=ctx, threads=8, tag="11,500 ppm")
    ctx.close()
    assert all(p == [0, 0, 0] for p in paths[-3:]), paths


def test_row_sparse_layer_at_a_warmup_density_stops_missing(rgc, oracle):
    """One row in twenty carries ten times larger values and overfills the tiles' lists on every call: after three misses on end
    the call takes the general launches, where a miss costs the layer at least one call without its hint (1 + 3 + 20 / 2 at most,
    of 24 calls)."""
    g = np.random.default_rng(17)
    rows, cols = 1024, 512
    n = rows * cols
    held = g.permutation(rows)[: rows // 4]

    def fill(s, which):
        scale = np.zeros((rows, 1), np.float32)
        scale[which] = 10.0
        return ((g.standard_normal((rows, cols)) * s).astype(np.float32) * scale).reshape(n)

    V = [fill(5e-3, held)]
    G_list = [[fill(1e-3, g.permutation(held)[: rows // 20])] for _ in range(24)]
    paths = run_iterations(rgc, oracle, V, G_list, [rgc.rgc_k_for_density(n, 20_000)], tag="row-sparse")
    assert paths[1:4] == [[2], [2], [2]], paths       # (the case is the one described)
    assert sum(p == [2] for p in paths) <= 14, paths


def test_hint_after_a_miss_is_aimed_like_one_after_a_hit(rgc):
    """A layer that is a dense one in the general launches, which derive its hint after a miss, and has lists in a tiled call: the
    candidates of a call after a miss are those of a call after a hit but for the noise of one gradient.  (The dense layer's aim, rank
    3 k in the place of 2.5 k, leaves a third more of them when the k sent are gone: the bound is half of that.)"""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(18)
    n = 2_000_000
    k = rgc.rgc_k_for_density(n, 15_625)
    V = torch.empty(n, device="cuda").normal_(0.0, 5e-3, generator=gen)
    G = torch.empty(n, device="cuda")
    oi = torch.empty(k, dtype=torch.int32, device="cuda")
    ov = torch.empty(k, dtype=torch.float32, device="cuda")
    oc = torch.zeros(1, dtype=torch.int32, device="cuda")
    layers = rgc.LayerList([G], [V], [k], [oi], [ov], oc)
    ctx = rgc.Context(n, 1)

    def step():
        G.normal_(0.0, 1e-3, generator=gen)
        rgc.rgc_compress_layers(ctx, layers, 0.0, 0, torch.cuda.current_stream())
        return ctx.last_stats(1)[0]

    for _ in range(12):
        after_hit = step()
    assert after_hit[0] == 0
    ctx.poison_hints(0)
    assert step()[0] == 2
    after_miss = step()
    assert after_miss[0] == 0
    assert abs(after_miss[1] - after_hit[1]) < 0.15 * after_hit[1], (after_hit, after_miss)
    ctx.close()


@pytest.mark.parametrize("velocity,path", [(False, 0), (True, 1)])
def test_layer_that_sends_many_of_very_many_elements(rgc, velocity, path):
    """720,000 of 240 million entries: without a velocity the layer is on the one-pass path, with one it is a dense layer, which has
    no hint where the optional scratch is not to be had.  The results are those of calls without hints."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(19)
    n, k = 240_000_000, 720_000
    G = torch.empty(n, device="cuda")

    def buffers():
        oi = torch.empty(k, dtype=torch.int32, device="cuda")
        ov = torch.empty(k, dtype=torch.float32, device="cuda")
        oc = torch.zeros(1, dtype=torch.int32, device="cuda")
        V = torch.empty(n, device="cuda").normal_(0.0, 5e-3, generator=gen)
        U = torch.empty(n, device="cuda").normal_(0.0, 1e-3, generator=gen) if velocity else None
        return V, U, oi, ov, oc

    sides = [buffers(), buffers()]
    sides[1][0].copy_(sides[0][0])
    if velocity:
        sides[1][1].copy_(sides[0][1])
    lists = [rgc.LayerList([G], [V], [k], [oi], [ov], oc, [U] if velocity else None) for V, U, oi, ov, oc in sides]
    ctxs = [rgc.Context(n, 1), rgc.Context(n, 1)]
    ctxs[0].limit_optional_scratch(0)
    paths = []
    for _ in range(6):
        G.normal_(0.0, 1e-3, generator=gen)
        for ctx, layers, flags in zip(ctxs, lists, (0, rgc.RGC_NO_HINTS)):
            rgc.rgc_compress_layers(ctx, layers, 0.9, flags, torch.cuda.current_stream())
        paths.append(ctxs[0].last_paths(1)[0])
        for name, a, b in zip(("residual", "velocity", "indices", "values", "count"), *sides):
            assert a is None or torch.equal(a.view(torch.int32), b.view(torch.int32)), name
    assert paths.count(path) >= (5 if path == 1 else 2) and paths[0] == 1, paths
    for ctx in ctxs:
        ctx.close()


def test_large_values_in_one_part_keep_their_hints(rgc, oracle):
    """The frequent rows of an embedding come first: nearly all candidates of a layer of seven parts lie in the first of them,
    more than one step holds, though no list runs over."""
    g = np.random.default_rng(13)
    n, ppm = (6 << 20) + 12_345, 1000
    k = rgc.rgc_k_for_density(n, ppm)
    scale = np.full(n, 1e-3, np.float32)
    scale[: n // 10] = 1.0
    V = [(g.standard_normal(n).astype(np.float32) * scale)]
    G_list = [[(g.standard_normal(n).astype(np.float32) * scale * 0.2)] for _ in range(8)]
    paths = run_iterations(rgc, oracle, V, G_list, [k], threads=8, tag="one part")
    assert all(p == [0] for p in paths[-4:]), paths


@pytest.mark.parametrize("ppm", [2000, 4000])
def test_large_values_in_whole_tiles_keep_their_hints(rgc, oracle, ppm):
    """The rows of an embedding that carry gradients: one stretch of 8192 elements in fifteen (seven) holds the large values, and
    a tile inside it has about 300 candidates, more than a sixteenth of its elements."""
    g = np.random.default_rng(15)
    n = (2 << 20) + 999
    scale = np.full(n, 1e-3, np.float32)
    every = 15 if ppm == 2000 else 7
    for at in range(0, n, every * 8192):
        scale[at:at + 8192] = 1.0
    V = [(g.standard_normal(n).astype(np.float32) * scale)]
    G_list = [[(g.standard_normal(n).astype(np.float32) * scale * 0.2)] for _ in range(8)]
    paths = run_iterations(rgc, oracle, V, G_list, [rgc.rgc_k_for_density(n, ppm)], threads=8, tag="whole tiles")
    assert all(p == [0] for p in paths[-4:]), paths


def test_missed_hints_take_the_fallback(rgc, oracle):
    """Hints too high, too low and random, heavy ties, an overflowing list, zeros: several layers at once go through the
    digits in the last launch, others do not."""
    g = np.random.default_rng(9)
    sizes = [300_000, 4_500_000, 40_001, 90_000, 400_000, 5000]
    V = [(g.standard_normal(n) * 1e-2).astype(np.float32) for n in sizes]
    V[2] = (np.round(V[2] * 300) / 300).astype(np.float32)
    V[3][:] = 0.0
    V[4][1000:2000] *= 100.0                                   # the 1000 largest, the rank aimed at, in one list of 480 slots
    G_list = [[(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] for _ in range(8)]
    for G in G_list:
        G[2] = (np.round(G[2] * 300) / 300).astype(np.float32)
        G[3][:] = 0.0
        G[4][1000:2000] *= 100.0
    ks = [rgc.rgc_k_for_density(n) for n in sizes]
    paths = run_iterations(rgc, oracle, V, G_list, ks, poison=[0, 1, 2, 2, 0, 1, 2], threads=8, tag="fallback")
    assert any(p[0] == 2 for p in paths) and any(p[1] == 2 for p in paths), paths


def test_alternating_selection(rgc, oracle):
    g = np.random.default_rng(10)
    sizes = [120_000, 33_000, 32_768, 700, 9]
    V0 = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
    V0[1][:] = np.abs(V0[1])                                    # no negative elements at first
    V0[2][:] = 0.0
    ks = [rgc.rgc_k_for_density(n) for n in sizes[:3]] + [200, 9]
    ctx = rgc.Context(sum(sizes), len(sizes))
    dev = GpuLayers(rgc, V0, ks)
    Vh = [v.copy() for v in V0]
    for t in range(6):
        G = [(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes]
        dev.set_grads(G)
        dev.step(ctx, 0.0, rgc.RGC_SELECT_SMALLEST if t % 2 else rgc.RGC_SELECT_LARGEST)
        idx, val, cnt, V, _ = dev.results()
        for l, n in enumerate(sizes):
            a = (Vh[l] + G[l]).astype(np.float32)
            order = np.argsort(a if t % 2 else -a, kind="stable")[: ks[l]]
            want = np.sort(order)
            assert np.array_equal(idx[l], want), "step %d layer %d" % (t, l)
            assert np.array_equal(u32(val[l]), u32(a[want])) and int(cnt[l]) == ks[l]
            a[want] = 0.0
            assert np.array_equal(u32(V[l]), u32(a))
            Vh[l] = a
    ctx.last_error()
    ctx.close()


def test_replayed_from_a_graph_with_misses(rgc, oracle):
    """The call recorded once and replayed; between the replays the hints are spoilt, so the fallback runs in some."""
    import torch
    g = np.random.default_rng(11)
    sizes = [200_000, 50_000, 1000]
    ks = [rgc.rgc_k_for_density(n) for n in sizes]
    V0 = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
    dev = GpuLayers(rgc, V0, ks)
    ctx = rgc.Context(sum(sizes), len(sizes))
    Vh = [v.copy() for v in V0]
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        graph = None
        for t in range(7):
            G = [(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes]
            dev.set_grads(G)
            if t in (3, 5):
                ctx.poison_hints(t % 3, s)
            if t < 2:
                rgc.rgc_compress_layers(ctx, dev.layers, 0.0, 0, s)
            else:
                if graph is None:
                    s.synchronize()
                    graph = torch.cuda.CUDAGraph()
                    with torch.cuda.graph(graph, stream=s):
                        rgc.rgc_compress_layers(ctx, dev.layers, 0.0, 0, s)
                graph.replay()
            s.synchronize()
            msgs = oracle_step(oracle, G, Vh, ks)
            assert_layers_equal("step %d" % t, ks, dev.results(), msgs, Vh)
            if t in (3, 5):
                assert 2 in ctx.last_paths(len(sizes), s)
    ctx.last_error(s)
    ctx.close()


def test_missed_hints_on_several_streams_at_once(rgc, oracle):
    """Six contexts, a thread and a stream each, all hints spoilt before every other call: the launches that put the missed
    layers right run beside each other and share the device."""
    import threading
    import torch
    sizes = [2_500_000, 300_000, 70_001, 4000]
    ks = [rgc.rgc_k_for_density(n) for n in sizes]
    steps, failed = 6, []
    inputs = []
    for c in range(6):
        g = np.random.default_rng(100 + c)
        inputs.append(([(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes],
                       [[(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] for _ in range(steps)]))
    contexts = [rgc.Context(sum(sizes), len(sizes)) for _ in inputs]
    devs = []
    for V0, _ in inputs:
        devs.append(GpuLayers(rgc, V0, ks))
    grads = [[[torch.from_numpy(g).cuda() for g in G] for G in Gs] for _, Gs in inputs]
    torch.cuda.synchronize()

    def work(c):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for t in range(steps):
                    for l in range(len(sizes)):
                        devs[c].G[l].copy_(grads[c][t][l])
                    if t % 2:
                        contexts[c].poison_hints(0, s)
                    rgc.rgc_compress_layers(contexts[c], devs[c].layers, 0.0, 0, s)
            s.synchronize()
            contexts[c].last_error(s)
            assert contexts[c].last_paths(len(sizes), s)[0] == 2
        except Exception as e:                                  # noqa: BLE001 (told to the test's own thread)
            failed.append((c, repr(e)))

    threads = [threading.Thread(target=work, args=(c,)) for c in range(len(inputs))]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not failed, failed
    for c, (V0, Gs) in enumerate(inputs):
        Vh = [v.copy() for v in V0]
        for G in Gs:
            msgs = oracle_step(oracle, G, Vh, ks, threads=8)
        assert_layers_equal("context %d" % c, ks, devs[c].results(), msgs, Vh)
        contexts[c].close()
