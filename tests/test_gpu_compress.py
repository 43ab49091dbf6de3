"""GPU parity: rgc_compress_layers (through the C ABI) against the CPU oracle, bit for bit on
indices, values, count, residual and velocity."""
import numpy as np
import pytest

from paper_1808_04357_amd import synth
from rgc_testutil import GpuLayers, assert_layers_equal, check_properties, oracle_step, u32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rgc():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1808_04357_amd as pkg
    pkg.load_library()
    return pkg


def run_iterations(rgc, oracle, V0, G_list, ks, U0=None, m=0.0, flags=0, ctx=None, misalign=0,
                   poison=None, tag="", threads=4, expect_paths=None):
    """Runs len(G_list) compression steps on both sides and compares after every step."""
    total = sum(v.size for v in V0)
    own = ctx is None
    if own:
        ctx = rgc.Context(total, len(V0))
    dev = GpuLayers(rgc, V0, ks, U0, misalign=misalign)
    Vh = [v.copy() for v in V0]
    Uh = [u.copy() for u in U0] if U0 is not None else None
    paths = []
    for t, G in enumerate(G_list):
        print("  %s step %d" % (tag, t), flush=True)
        if poison is not None and t > 0:
            ctx.poison_hints(poison[(t - 1) % len(poison)])
        dev.set_grads(G)
        dev.step(ctx, m, flags)
        msgs = oracle_step(oracle, G, Vh, ks, Uh, m, mask_momentum=not (flags & rgc.RGC_NO_MOMENTUM_MASK),
                           threads=threads, nesterov=bool(flags & rgc.RGC_NESTEROV))
        assert_layers_equal("%s step %d" % (tag, t), ks, dev.results(), msgs, Vh, Uh)
        paths.append(ctx.last_paths(len(V0)))
    if expect_paths is not None:
        expect_paths(paths)
    if own:
        ctx.close()
    return paths


def test_wave_primitives_selftest(rgc):
    ctx = rgc.Context(1024, 1)
    ctx.selftest()
    ctx.close()


def test_config1_single_layer_five_steps(rgc, oracle):
    cfg = synth.config_single(1 << 20, num_grads=5)
    ks = [rgc.rgc_k_for_density(1 << 20)]
    assert ks == [1049]

    def expect(paths):
        assert paths[0] == [1], "first call has no hint"
        assert all(p == [0] for p in paths[1:]), "later calls take the one-pass path: %r" % (paths,)

    run_iterations(rgc, oracle, cfg["V"], cfg["G"], ks, tag="C1", expect_paths=expect)


@pytest.mark.parametrize("flags_name", ["default", "no_hints"])
def test_ragged_sizes_batched(rgc, oracle, flags_name):
    sizes = [1, 2, 3, 63, 64, 65, 255, 256, 257, 1000, 4096, 8191, 8192, 8193, 3 * 8192 + 5,
             100_003, 4 * 8192, 262_147]
    g = np.random.default_rng(42)
    V = [(g.standard_normal(n) * 1e-2).astype(np.float32) for n in sizes]
    ks = []
    for i, n in enumerate(sizes):
        ks.append([1, n, max(1, n // 2), rgc.rgc_k_for_density(n), max(1, n // 10)][i % 5])
    G_list = [[(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] for _ in range(4)]
    flags = rgc.RGC_NO_HINTS if flags_name == "no_hints" else 0
    run_iterations(rgc, oracle, V, G_list, ks, flags=flags, tag="ragged-" + flags_name)


def test_unaligned_tensors(rgc, oracle):
    sizes = [5, 300, 8192 + 7, 50_001]
    g = np.random.default_rng(43)
    V = [(g.standard_normal(n)).astype(np.float32) for n in sizes]
    U = [(g.standard_normal(n)).astype(np.float32) for n in sizes]
    ks = [2, 3, 9, 51]
    G_list = [[(g.standard_normal(n) * 0.1).astype(np.float32) for n in sizes] for _ in range(3)]
    for mis in (1, 2, 3):
        run_iterations(rgc, oracle, V, G_list, ks, U0=U, m=0.9, misalign=mis, tag="misalign%d" % mis)


def test_ties_zeros_and_constant_tensors(rgc, oracle):
    g = np.random.default_rng(44)
    n = 70_000
    quant = (np.round(g.standard_normal(n) * 4) / 4).astype(np.float32)       # ~20 distinct magnitudes
    V = [quant, np.zeros(n, np.float32), np.full(n, -2.5, np.float32), np.zeros(9000, np.float32),
         np.where(np.arange(n) % 7 == 0, 1.0, -1.0).astype(np.float32)]
    ks = [700, 70, 123, 9000, 33]
    zero = [np.zeros(v.size, np.float32) for v in V]
    small = [(np.round(g.standard_normal(v.size)) * 0.25).astype(np.float32) for v in V]
    run_iterations(rgc, oracle, V, [zero, small, zero, small, small], ks, tag="ties")


def test_nan_inf_denormal(rgc, oracle):
    g = np.random.default_rng(45)
    n = 20_000
    V = (g.standard_normal(n) * 1e-3).astype(np.float32)
    V[[5, 77, 9000]] = [np.nan, np.inf, -np.inf]
    V[100:200] = np.float32(1e-41)       # denormals must survive the add and order correctly
    V[300:400] = np.float32(-3e-42)
    G = np.zeros(n, np.float32)
    G[150] = np.float32(2e-41)
    G2 = (g.standard_normal(n) * 1e-42).astype(np.float32)
    run_iterations(rgc, oracle, [V], [[G], [G2], [G2]], [40], tag="special")
    # a layer of denormals only: selection must order them by magnitude
    Vd = (g.integers(-2000, 2000, n).astype(np.float64) * 1.4e-45).astype(np.float32)
    run_iterations(rgc, oracle, [Vd], [[G2], [G2]], [25], tag="denormal")


@pytest.mark.parametrize("mask", [True, False])
def test_momentum_variant(rgc, oracle, mask):
    g = np.random.default_rng(46)
    sizes = [40_000, 9000, 130]
    V = [(g.laplace(0, 5e-3, n)).astype(np.float32) for n in sizes]
    U = [(g.laplace(0, 1e-3, n)).astype(np.float32) for n in sizes]
    ks = [rgc.rgc_k_for_density(n) for n in sizes]
    G_list = [[(g.laplace(0, 1e-3, n)).astype(np.float32) for n in sizes] for _ in range(4)]
    flags = 0 if mask else rgc.RGC_NO_MOMENTUM_MASK
    run_iterations(rgc, oracle, V, G_list, ks, U0=U, m=0.9, flags=flags, tag="momentum-mask%d" % mask)


def test_results_do_not_depend_on_hints(rgc, oracle):
    """Poisoned thresholds (too high, too low, random) must only cost time."""
    cfg = synth.config_single(300_000, num_grads=7)
    g = np.random.default_rng(47)
    sizes = [300_000, 50_000, 2048, 64]
    V = [cfg["V"][0]] + [(g.standard_normal(n) * 1e-2).astype(np.float32) for n in sizes[1:]]
    G_list = [[cfg["G"][t][0]] + [(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes[1:]]
              for t in range(7)]
    ks = [rgc.rgc_k_for_density(n) for n in sizes]
    paths = run_iterations(rgc, oracle, V, G_list, ks, poison=[0, 1, 2, 2, 0, 1], tag="poison")
    assert any(p != 0 for step in paths[1:] for p in step), "poisoned hints should force fallbacks"


def test_hint_signature_change_and_reuse_of_context(rgc, oracle):
    g = np.random.default_rng(48)
    ctx = rgc.Context(200_000, 4)
    for sizes in ([100_000, 777], [90_000, 777, 5000], [100_000, 777]):
        V = [(g.standard_normal(n) * 1e-2).astype(np.float32) for n in sizes]
        G_list = [[(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] for _ in range(3)]
        ks = [rgc.rgc_k_for_density(n) for n in sizes]
        run_iterations(rgc, oracle, V, G_list, ks, ctx=ctx, tag="reuse%d" % len(sizes))
    ctx.reset_hints()
    ctx.close()


def test_uniform_distribution_of_the_papers_selection_benchmark(rgc, oracle):
    cfg = synth.config_uniform(1 << 21, num_grads=3)
    ks = [rgc.rgc_k_for_density(1 << 21)]
    run_iterations(rgc, oracle, cfg["V"], cfg["G"], ks, tag="uniform")


def test_larger_density(rgc, oracle):
    """Warm-up densities (Section 2.5 lists 25 % ... 0.1 %) must be correct for any k."""
    g = np.random.default_rng(49)
    n = 200_000
    for ppm in (250_000, 62_500, 15_625, 4_000):
        V = [(g.standard_normal(n) * 1e-2).astype(np.float32)]
        G_list = [[(g.standard_normal(n) * 1e-3).astype(np.float32)] for _ in range(2)]
        run_iterations(rgc, oracle, V, G_list, [rgc.rgc_k_for_density(n, ppm)], tag="ppm%d" % ppm)


@pytest.mark.parametrize("ppm", [250_000, 62_500, 15_625])
@pytest.mark.parametrize("variant", ["plain", "momentum", "nesterov_unmasked"])
def test_warmup_densities_take_the_dense_path(rgc, oracle, ppm, variant):
    """Section 2.5's warm-up densities on layers of several wave-chunks: the first call is hint-free, later
    calls list every candidate while they stream, mask those above the expected k-th key at once and put right
    what that got wrong when the message is written; every step bit for bit."""
    g = np.random.default_rng(500 + ppm % 97)
    sizes = [300_000, 70_001, 40_960, 9_000]
    # gradients larger than the residual: the k-th magnitude then hardly moves from call to call, as in
    # steady training (with a residual that only drains, it moves by a whole k ranks per call and no
    # narrow band around the last threshold can hold the next one)
    # (the velocity starts at its stationary scale for the same reason)
    V = [(g.laplace(size=n) * 1e-3).astype(np.float32) for n in sizes]
    U = [(g.laplace(size=n) * 1.15e-2).astype(np.float32) for n in sizes] if variant != "plain" else None
    G_list = [[(g.laplace(size=n) * 1e-2).astype(np.float32) for n in sizes] for _ in range(14)]
    ks = [rgc.rgc_k_for_density(n, ppm) for n in sizes]
    flags = (rgc.RGC_NESTEROV | rgc.RGC_NO_MOMENTUM_MASK) if variant == "nesterov_unmasked" else 0

    def expect(paths):
        assert all(p == 1 for p in paths[0]), "first call has no hint"
        assert any(step[0] == 0 for step in paths[1:]), "the large layer never left the multi-pass path: %r" % (paths,)

    run_iterations(rgc, oracle, V, G_list, ks, U0=U, m=0.5 if U is not None else 0.0, flags=flags,
                   tag="warmup %d ppm %s" % (ppm, variant), expect_paths=expect)


def test_dense_layers_with_poisoned_hints_ties_and_unaligned_tensors(rgc, oracle):
    """The streaming pass of a dense layer must notice a useless hint (too high, too low, random), heavy ties (the
    bin of the k-th key does not fit the ranking) and list overflows, put back what it masked on the strength of the
    hint, and the call must still give the exact result."""
    g = np.random.default_rng(77)
    sizes = [200_003, 131_072, 60_000]
    ks = [rgc.rgc_k_for_density(n, 62_500) for n in sizes]
    V = [(g.standard_normal(n) * 1e-2).astype(np.float32) for n in sizes]
    V[1] = (np.round(V[1] * 800) / 800).astype(np.float32)                     # a few dozen distinct magnitudes
    G_list = [[(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] for _ in range(7)]
    for G in G_list:
        G[1][:] = (np.round(G[1] * 800) / 800).astype(np.float32)
    paths = run_iterations(rgc, oracle, V, G_list, ks, poison=[0, 1, 2, 2, 0, 1], misalign=1, tag="dense poison")
    assert any(p == 2 for step in paths[1:] for p in step), "poisoned hints should make the hinted pass miss: %r" % (paths,)


def test_dense_layers_clustered_values_overflow_single_lists(rgc, oracle):
    """All large values in one stretch of the tensor: the lists of those wave-chunks run over, the pass stops listing
    and masking there, and what it had masked by then is put back."""
    g = np.random.default_rng(78)
    n = 400_000
    ks = [rgc.rgc_k_for_density(n, 62_500)]
    scale = np.full(n, 1e-4, np.float32)
    scale[100_000:130_000] = 1.0
    V = [(g.standard_normal(n).astype(np.float32) * scale)]
    G_list = [[(g.standard_normal(n).astype(np.float32) * scale * 0.1)] for _ in range(4)]
    run_iterations(rgc, oracle, V, G_list, ks, tag="dense clustered")


def test_dense_layers_without_their_scratch_take_the_hint_free_path(rgc, oracle):
    """The lists of the dense layers are allocated on demand; when they cannot be had (here: capped to nothing) the
    layers take the hint-free path call after call and the results are the same; with the cap lifted the same
    context goes on to the hinted path."""
    g = np.random.default_rng(81)
    sizes = [300_000, 40_960]
    ks = [rgc.rgc_k_for_density(n, 62_500) for n in sizes]
    V = [(g.laplace(size=n) * 1e-3).astype(np.float32) for n in sizes]
    G_list = [[(g.laplace(size=n) * 1e-2).astype(np.float32) for n in sizes] for _ in range(10)]
    ctx = rgc.Context(sum(sizes), len(sizes))
    ctx.limit_optional_scratch(0)
    dev = GpuLayers(rgc, V, ks)
    Vh = [v.copy() for v in V]
    paths = []
    for t, G in enumerate(G_list):
        if t == 4:
            ctx.limit_optional_scratch(-1)
        dev.set_grads(G)
        dev.step(ctx, 0.0, 0)
        msgs = oracle_step(oracle, G, Vh, ks)
        assert_layers_equal("capped scratch step %d" % t, ks, dev.results(), msgs, Vh)
        paths.append(ctx.last_paths(len(sizes)))
    assert all(p == [1, 1] for p in paths[:4]), paths
    assert any(p[0] == 0 for p in paths[4:]), paths
    ctx.last_error()
    ctx.close()


def test_dense_layer_whose_kth_key_is_a_long_tie(rgc, oracle):
    """The k-th key is shared by more than a thousand elements, call after call, and they sit in five wave-chunks of two
    workgroups whose members go to the same sub-list: the streaming pass masks them all (their key is the expected k-th
    key), the ranking takes more members than that sub-list holds, the lowest indices win, and the output step puts the
    others back."""
    g = np.random.default_rng(79)
    n, k = 400_000, 25_000
    per_step = 100
    c = np.float32(0.25)
    # 300 tied elements in each of the wave-chunks 4, 5, 6, 7 and 69 (of 4096 elements): workgroups 1 and 17 of the layer
    tie = np.concatenate([np.arange(w * 4096 + 7, w * 4096 + 307) for w in (4, 5, 6, 7, 69)])
    rest = np.setdiff1d(np.arange(n), tie)
    large = np.sort(g.choice(rest, size=k - per_step, replace=False))   # sent on every call, and large again on the next
    V = np.zeros(n, np.float32)
    V[rest] = (g.standard_normal(rest.size) * 1e-2).astype(np.float32)  # well below the tied value
    V[tie] = c
    V[tie[::7]] = -c                                                    # the tie is one of magnitudes
    V[large] = 0.0
    G_list = []
    for _ in range(9):
        G = np.zeros(n, np.float32)
        G[large] = (1.0 + g.random(large.size)).astype(np.float32) * g.choice([-1.0, 1.0], size=large.size).astype(np.float32)
        G_list.append([G])
    paths = run_iterations(rgc, oracle, [V], G_list, [k], tag="dense tie")
    assert sum(1 for p in paths[1:] if p == [0]) >= 4, "the hinted path of the dense layer was hardly taken: %r" % (paths,)


@pytest.mark.parametrize("ties", [1_900, 2_100, 3_500])
def test_sparse_layer_beside_a_dense_one_whose_kth_key_is_a_long_tie(rgc, oracle, ties):
    """Calls with a dense layer rank the members of the other layers' coarse bins in a smaller share of the LDS (2048
    members) and longer ties where they are: the k-th key of the second layer is shared by up to 3500 elements."""
    g = np.random.default_rng(82)
    n, k, per_step = 400_000, 2_000, 20
    tie = np.sort(g.choice(n, size=ties, replace=False))
    rest = np.setdiff1d(np.arange(n), tie)
    large = np.sort(g.choice(rest, size=k - per_step, replace=False))   # sent on every call, and large again on the next
    V = [(g.standard_normal(100_000) * 1e-2).astype(np.float32), (g.standard_normal(n) * 1e-2).astype(np.float32)]
    V[1][tie] = 0.25
    V[1][large] = 0.0
    G_list = []
    for _ in range(5):
        G = np.zeros(n, np.float32)
        G[large] = (1.0 + g.random(large.size)).astype(np.float32)
        G_list.append([(g.standard_normal(100_000) * 1e-3).astype(np.float32), G])
    paths = run_iterations(rgc, oracle, V, G_list, [rgc.rgc_k_for_density(100_000, 62_500), k], tag="%d ties" % ties)
    assert sum(1 for p in paths[1:] if p == [0, 0]) >= 2, paths


def test_output_steps_from_either_end_beside_layers_whose_hint_missed(rgc, oracle):
    """A dense call that writes more than the memory-side cache holds, with the largest layer, the other one or both on the five
    passes after a jump of the gradient."""
    g = np.random.default_rng(83)
    sizes = [33_600_000, 300_001]
    ks = [rgc.rgc_k_for_density(n, 20_000) for n in sizes]
    V = [(g.standard_normal(n, dtype=np.float32) * np.float32(1e-2)) for n in sizes]
    U = [(g.standard_normal(n, dtype=np.float32) * np.float32(1e-3)) for n in sizes]
    base = [(g.standard_normal(n, dtype=np.float32) * np.float32(1e-3)) for n in sizes]
    G_list = []
    for first, second in [(1, 1), (1, 1), (1, 1), (1, 1), (300, 1), (1, 1), (1, 1), (1, 1), (1, 300), (1, 1), (1, 1)]:
        G_list.append([b * np.float32(f) for b, f in zip(base, (first, second))])
    paths = run_iterations(rgc, oracle, V, G_list, ks, U0=U, m=0.9, threads=16, tag="either end")
    assert paths[4][0] == 2 and paths[8][1] == 2, paths        # (the jumps miss)
    assert any(p[0] == 0 for p in paths) and any(p[1] == 0 for p in paths), paths


@pytest.mark.parametrize("ppm", [250_000, 15_625])
def test_config3_vgg16_set_full_size_warmup_density(rgc, oracle, ppm):
    """The VGG16-shaped set with the momentum correction at a warm-up density, at full size (the configuration
    the benchmark's warm-up block times).  The threshold hints of the dense layers need a few calls to settle
    (the first hinted call finds the residual's k-th magnitude far from where the hint-free call left it), so
    eight calls run on the GPU alone; the oracle then starts from the residual and velocity the GPU holds and
    the next two calls are compared bit for bit, with the large layers on their hinted path."""
    cfg = synth.config_vgg16(num_grads=4)
    V0, U0, G_list, m = cfg["V"], cfg["U"], cfg["G"], cfg["momentum"]
    ks = [rgc.rgc_k_for_density(v.size, ppm) for v in V0]
    ctx = rgc.Context(sum(v.size for v in V0), len(V0))
    dev = GpuLayers(rgc, V0, ks, U0)
    for t in range(8):
        dev.set_grads(G_list[t % 4])
        dev.step(ctx, m, 0)
    _, _, _, Vh, Uh = dev.results()
    paths = []
    for t in range(8, 10):
        print("  C3 %d ppm step %d" % (ppm, t), flush=True)
        G = G_list[t % 4]
        dev.set_grads(G)
        dev.step(ctx, m, 0)
        msgs = oracle_step(oracle, G, Vh, ks, Uh, m, threads=16)
        assert_layers_equal("C3 %d ppm step %d" % (ppm, t), ks, dev.results(), msgs, Vh, Uh)
        paths.append(ctx.last_paths(len(V0)))
    big = int(np.argmax([v.size for v in V0]))
    assert any(p[big] == 0 for p in paths), "the largest layer never took its hinted path: %r" % (paths,)
    ctx.close()


def test_config4_lstm_set_full_size_warmup_density(rgc, oracle):
    """The LSTM-shaped set at full size at 6.25 %: the embedding tensor is three quarters zeros (row-sparse gradient
    and residual), the layers are dense ones and reach their hinted path within a few calls."""
    cfg = synth.config_lstm(num_grads=4)
    ks = [rgc.rgc_k_for_density(v.size, 62_500) for v in cfg["V"]]
    G_list = [cfg["G"][t % 4] for t in range(5)]
    paths = run_iterations(rgc, oracle, cfg["V"], G_list, ks, tag="C4 62500 ppm", threads=16)
    assert any(p.count(0) >= 5 for p in paths[1:]), "the dense layers never took their hinted path: %r" % (paths,)


def test_config2_resnet50_set(rgc, oracle):
    cfg = synth.config_resnet50(num_grads=3)
    ks = [rgc.rgc_k_for_density(v.size) for v in cfg["V"]]
    assert len(ks) == 161 and sum(ks) == 25_670
    run_iterations(rgc, oracle, cfg["V"], cfg["G"], ks, tag="C2", threads=16)


def test_config4_lstm_set_full_size(rgc, oracle):
    cfg = synth.config_lstm(num_grads=2)
    ks = [rgc.rgc_k_for_density(v.size) for v in cfg["V"]]
    assert sum(ks) == 66_024
    run_iterations(rgc, oracle, cfg["V"], cfg["G"], ks, tag="C4", threads=16)


def test_config3_vgg16_set_full_size_momentum(rgc, oracle):
    cfg = synth.config_vgg16(num_grads=2)
    ks = [rgc.rgc_k_for_density(v.size) for v in cfg["V"]]
    assert sum(ks) == 138_351
    run_iterations(rgc, oracle, cfg["V"], cfg["G"], ks, U0=cfg["U"], m=cfg["momentum"], tag="C3", threads=16)


def test_argument_errors(rgc):
    import torch
    ctx = rgc.Context(10_000, 2)
    dev = torch.device("cuda:0")
    g = torch.zeros(100, device=dev)
    v = torch.zeros(100, device=dev)
    oi = torch.zeros(10, dtype=torch.int32, device=dev)
    ov = torch.zeros(10, device=dev)
    oc = torch.zeros(4, dtype=torch.int32, device=dev)

    def status(fn):
        with pytest.raises(rgc.RgcError) as e:
            fn()
        return e.value.status

    ok = rgc.LayerList([g], [v], [10], [oi], [ov], oc)
    rgc.rgc_compress_layers(ctx, ok)
    assert status(lambda: rgc.rgc_compress_layers(ctx, rgc.LayerList([g], [v], [0], [oi], [ov], oc))) == -1
    assert status(lambda: rgc.rgc_compress_layers(ctx, rgc.LayerList([g], [v], [101], [oi], [ov], oc))) == -1
    assert status(lambda: rgc.rgc_compress_layers(ctx, ok, flags=0x80)) == -1
    three = rgc.LayerList([g, g, g], [v, v, v], [1, 1, 1], [oi, oi, oi], [ov, ov, ov], oc)
    assert status(lambda: rgc.rgc_compress_layers(ctx, three)) == -1            # more layers than the context
    big = torch.zeros(20_000, device=dev)
    assert status(lambda: rgc.rgc_compress_layers(
        ctx, rgc.LayerList([big], [big.clone()], [1], [oi], [ov], oc))) == -2    # scratch too small
    bad = rgc.LayerList([g], [v], [10], [oi], [ov], oc)
    bad.array[0].residual = None
    assert status(lambda: rgc.rgc_compress_layers(ctx, bad)) == -1
    torch.cuda.synchronize()
    ctx.close()


def test_two_contexts_on_two_streams(rgc, oracle):
    """Two contexts used on two streams at once (calls of the two interleaved, nothing between them
    synchronised): each must give its own layer set's oracle result on every step."""
    import torch
    g = np.random.default_rng(52)
    sets = []
    for s, sizes in enumerate([[300_000, 70_000, 5_000], [1 << 20]]):
        V = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
        Gs = [[(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] for _ in range(4)]
        ks = [rgc.rgc_k_for_density(n) for n in sizes]
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            dev = GpuLayers(rgc, V, ks)
        sets.append(dict(V=[v.copy() for v in V], Gs=Gs, ks=ks, dev=dev, stream=stream,
                         ctx=rgc.Context(sum(sizes), len(sizes))))
    torch.cuda.synchronize()
    for t in range(4):
        for S in sets:                                   # enqueue on both streams before looking at either
            with torch.cuda.stream(S["stream"]):
                S["dev"].set_grads(S["Gs"][t])
            rgc.rgc_compress_layers(S["ctx"], S["dev"].layers, 0.0, 0, S["stream"])
        for s, S in enumerate(sets):
            S["stream"].synchronize()
            msgs = oracle_step(oracle, S["Gs"][t], S["V"], S["ks"])
            assert_layers_equal("stream %d step %d" % (s, t), S["ks"], S["dev"].results(), msgs, S["V"])
    for S in sets:
        S["ctx"].close()


def test_nesterov_form_of_the_momentum_correction(rgc, oracle):
    """RGC_NESTEROV: u = m (u + g), a = (V + u) + g, over several steps, with and without masking."""
    g = np.random.default_rng(61)
    sizes = [150_000, 33_333, 4097, 9]
    for flags in (rgc.RGC_NESTEROV, rgc.RGC_NESTEROV | rgc.RGC_NO_MOMENTUM_MASK):
        V = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
        U = [(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes]
        Gs = [[(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] for _ in range(5)]
        ks = [rgc.rgc_k_for_density(n) for n in sizes]
        run_iterations(rgc, oracle, V, Gs, ks, U0=U, m=0.9, flags=flags, tag="nesterov flags %d" % flags)
    # layers without a velocity ignore the flag
    V = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
    Gs = [[(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] for _ in range(2)]
    run_iterations(rgc, oracle, V, Gs, [rgc.rgc_k_for_density(n) for n in sizes], flags=rgc.RGC_NESTEROV, tag="no velocity")


def ulp_distance(a, b):
    ia = int(np.array(a, np.float32).view(np.int32))
    ib = int(np.array(b, np.float32).view(np.int32))
    return abs(ia - ib)


def test_clipping_coefficient_and_scaled_gradients(rgc, oracle):
    """rgc_clip_coefficient against the oracle's (both take the exactly rounded sum of the squares: bit for
    bit), then rgc_compress_layers_scaled with that very coefficient against the oracle fed the
    same number: bit for bit, several steps, plain, momentum-corrected and Nesterov."""
    import torch
    g = np.random.default_rng(62)
    sizes = [300_000, 70_001, 4096, 5]
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream()
    coef = torch.full((1,), float("nan"), dtype=torch.float32, device=dev)
    for m, flags, with_u in ((0.0, 0, False), (0.9, 0, True), (0.9, rgc.RGC_NESTEROV, True)):
        V = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
        U = [(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] if with_u else None
        ks = [rgc.rgc_k_for_density(n) for n in sizes]
        ctx = rgc.Context(sum(sizes), len(sizes))
        layers = GpuLayers(rgc, V, ks, U)
        Vh = [v.copy() for v in V]
        Uh = [u.copy() for u in U] if with_u else None
        for t in range(4):
            G = [(g.standard_normal(n) * (1e-3 * (1 + 3 * (t % 2)))).astype(np.float32) for n in sizes]
            layers.set_grads(G)
            max_norm = 4.0                             # threshold 4 / sqrt(16) = 1: exceeded on the odd steps only (norms 0.6 and 2.4)
            rgc.rgc_clip_coefficient(ctx, layers.layers, max_norm, 16, coef, stream)
            c_gpu = float(coef.cpu().numpy()[0])
            c_ref, sq = oracle.clip_coefficient(G, max_norm, 16)
            assert ulp_distance(c_gpu, c_ref) == 0, (t, c_gpu, c_ref)
            if t % 2 == 0:
                assert c_ref == 1.0 and c_gpu == 1.0, "below the threshold nothing is scaled"
            else:
                assert c_ref < 1.0
            layers.step(ctx, m, flags, grad_scale=coef)
            msgs = oracle_step(oracle, G, Vh, ks, Uh, m, nesterov=bool(flags & rgc.RGC_NESTEROV), grad_scale=c_gpu)
            assert_layers_equal("scaled m=%g flags=%d step %d" % (m, flags, t), ks, layers.results(), msgs, Vh, Uh)
        ctx.close()


@pytest.mark.parametrize("law", ["wide", "tiny_beside_large", "subnormal", "infinite", "nan"])
def test_clipping_coefficient_of_hard_norms(rgc, oracle, law):
    """Gradients whose squares span the whole fp64-exact range of fp32 products, tiny elements beside large
    ones (their squares fall below the last bit of a running fp64 sum), subnormal elements, and elements that
    are not finite (norm infinite: coefficient 0; norm NaN: the comparison fails, coefficient 1)."""
    import torch
    g = np.random.default_rng({"wide": 11, "tiny_beside_large": 12, "subnormal": 13, "infinite": 14, "nan": 15}[law])
    sizes = [100_003, 9_000, 300, 2]
    G = []
    for n in sizes:
        if law == "wide":
            x = g.standard_normal(n) * np.exp2(g.integers(-70, 55, n).astype(np.float64))
        elif law == "tiny_beside_large":
            x = g.standard_normal(n) * np.where(g.random(n) < 0.5, 1e-12, 1.0)
        elif law == "subnormal":
            x = g.integers(-2 ** 22, 2 ** 22, n).astype(np.float64) * 2.0 ** -149
        else:
            x = g.standard_normal(n)
        G.append(x.astype(np.float32))
    if law == "infinite":
        G[1][5] = -np.inf
    if law == "nan":
        G[2][5] = np.nan
        G[0][1] = np.inf
    V = [np.zeros(n, np.float32) for n in sizes]
    layers = GpuLayers(rgc, V, [1] * len(sizes))
    layers.set_grads(G)
    ctx = rgc.Context(sum(sizes), len(sizes))
    coef = torch.full((1,), 7.0, dtype=torch.float32, device=torch.device("cuda:0"))
    for max_norm, workers in ((1e-30, 4), (1.0, 16), (1e30, 1)):
        print("  hard norms: %s max_norm %g" % (law, max_norm), flush=True)
        rgc.rgc_clip_coefficient(ctx, layers.layers, max_norm, workers, coef, torch.cuda.current_stream())
        c_gpu = coef.cpu().numpy()[0]
        c_ref, sq = oracle.clip_coefficient(G, max_norm, workers)
        assert np.float32(c_gpu).view(np.uint32) == np.float32(c_ref).view(np.uint32), (law, max_norm, c_gpu, c_ref, sq)
    if law == "infinite":
        assert c_gpu == 0.0
    if law == "nan":
        assert c_gpu == 1.0
    ctx.close()


def test_clipping_coefficient_full_size_vgg16(rgc, oracle):
    import torch
    cfg = synth.config_vgg16(num_grads=1)
    G = cfg["G"][0]
    V = cfg["V"]
    ks = [rgc.rgc_k_for_density(v.size) for v in V]
    layers = GpuLayers(rgc, V, ks)
    layers.set_grads(G)
    ctx = rgc.Context(sum(v.size for v in V), len(V))
    coef = torch.zeros(1, dtype=torch.float32, device=torch.device("cuda:0"))
    rgc.rgc_clip_coefficient(ctx, layers.layers, 1.0, 128, coef, torch.cuda.current_stream())
    c_ref, sq = oracle.clip_coefficient(G, 1.0, 128)
    c_gpu = float(coef.cpu().numpy()[0])
    assert c_ref < 1.0 and ulp_distance(c_gpu, c_ref) == 0, (c_gpu, c_ref, sq)
    ctx.close()


def test_stream_yardstick_computes_the_bare_update(rgc):
    """The benchmark's yardstick kernel does the momentum-corrected accumulate and nothing else: compared with the two
    fp32 operations written out in numpy (no contraction on either side), ragged lengths, both directions."""
    import torch
    g = np.random.default_rng(90)
    for n in (1, 3, 4, 255, 8192, 8193, 4 * 8192 + 2, 100_003):
        G = (g.standard_normal(n) * 1e-3).astype(np.float32)
        V = (g.standard_normal(n) * 1e-2).astype(np.float32)
        U = (g.standard_normal(n) * 1e-3).astype(np.float32)
        m = np.float32(0.9)
        dg, dv, du = (torch.from_numpy(a).cuda() for a in (G, V, U))
        for t in range(2):
            print("  yardstick n %d call %d" % (n, t), flush=True)
            rgc.rgc_stream_yardstick(dg, dv, du, float(m), reverse=bool(t))
            U = (m * U).astype(np.float32) + G
            V = V + U
        torch.cuda.synchronize()
        assert np.array_equal(u32(du.cpu().numpy()), u32(U)) and np.array_equal(u32(dv.cpu().numpy()), u32(V)), n
    with pytest.raises(rgc.RgcError):
        rgc.rgc_stream_yardstick(dg[1:], dv[1:], du[1:], 0.9)          # not 16-byte aligned
