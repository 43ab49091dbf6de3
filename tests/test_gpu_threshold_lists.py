"""GPU parity of a searching threshold call where its lists do, and where they do not: layers at the sizes and densities
where the sample changes, values that fill single lists, sparse layers, searches that end below what was listed (bit equality)."""
import numpy as np
import pytest

from test_gpu_threshold import Runner

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rgc():
    import paper_1808_04357_amd as m
    return m


LINE = 8 << 20     # elements of a call from which it lists (kSampleElems)


@pytest.fixture(scope="module")
def filler():
    """A layer that takes its call to the line: residual, gradient, velocity."""
    g = np.random.default_rng(5)
    return [(g.standard_normal(LINE, dtype=np.float32) * np.float32(s)) for s in (5e-3, 1e-3, 1e-3)]


@pytest.mark.parametrize("ppm", [100, 1000, 7000, 9000, 100_000])
@pytest.mark.parametrize("momentum,nesterov", [(False, False), (True, False), (True, True)])
def test_densities_and_sample_sizes(rgc, oracle, filler, ppm, momentum, nesterov):
    g = np.random.default_rng(ppm)
    sizes = [3, 4095, 16383, 16385, 65_537, 1_000_003]
    ks = [rgc.rgc_k_for_density(n, ppm) for n in sizes]
    V = [(g.standard_normal(n) * 5e-3).astype(np.float32) for n in sizes]
    U = [(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] + [filler[2]] if momentum else None
    V.append(filler[0])
    ks.append(rgc.rgc_k_for_density(LINE, 1000))
    r = Runner(rgc, oracle, V, ks, U0=U, m=0.9, misalign=1, tag="threshold lists")
    for t in range(3):
        r.step([(g.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes] + [filler[1]], search=t != 1, nesterov=nesterov,
               grad_scale=0.5 if t == 2 else None)
    r.close()


@pytest.mark.parametrize("listed", [True, False])
@pytest.mark.parametrize("law", ["clustered", "row sparse", "nearly all zero", "two levels", "uniform", "one outlier"])
def test_layers_whose_lists_may_not_do(rgc, oracle, filler, law, listed):
    g = np.random.default_rng(17)
    n = 600_000
    k = rgc.rgc_k_for_density(n)

    def draw(s):
        a = (g.standard_normal(n) * s).astype(np.float32)
        if law == "clustered":
            a *= np.where((np.arange(n) > 50_000) & (np.arange(n) < 53_000), np.float32(100.0), np.float32(1.0))
        elif law == "row sparse":
            a.reshape(400, 1500)[g.permutation(400)[:380]] = 0.0
        elif law == "nearly all zero":
            a[g.permutation(n)[k // 2:]] = 0.0
        elif law == "two levels":
            a = np.where(g.random(n) < 0.003, np.float32(1.0), np.float32(0.25)).astype(np.float32) * np.float32(s)
        elif law == "uniform":
            a = (g.random(n) * s).astype(np.float32)
        else:
            a[7] = 1e4                                           # every threshold tried lies far above the others
        return a

    more = LINE if listed else LINE - n - 200_000 - 1           # at the line, and one element below it
    V = [draw(1.0), g.standard_normal(200_000).astype(np.float32), filler[0][:more]]
    r = Runner(rgc, oracle, V, [k, 200, more // 1000], tag="threshold " + law)
    for t in range(3):
        r.step([draw(0.05), (g.standard_normal(200_000) * 0.1).astype(np.float32), filler[1][:more]], search=True)
    r.close()


@pytest.mark.parametrize("clustered", [False, True])
@pytest.mark.parametrize("ppm", [30_000, 62_500, 250_000])
def test_small_lists_of_dense_layers(rgc, oracle, ppm, clustered):
    """Small calls that no tiled call can take: wave-chunks of 2048 elements with 128 slots each, which hold what lies above a reused
    threshold, or run over (everywhere at the higher densities, where the values sit together at all)."""
    g = np.random.default_rng(ppm + clustered)
    sizes = [2047, 2049, 8193, 300_001, 700_001]
    ks = [rgc.rgc_k_for_density(n, ppm) for n in sizes]

    def draw(s):
        a = [(g.standard_normal(n) * s).astype(np.float32) for n in sizes]
        if clustered:
            a = [x * np.where(g.random(-(-x.size // 2048)) < 0.1, np.float32(20.0), np.float32(1.0)).repeat(2048)[:x.size] for x in a]
        return a

    r = Runner(rgc, oracle, draw(1.0), ks, U0=draw(0.1), m=0.9, misalign=1, tag="threshold small")
    for search in (True, False, True, False):
        r.step(draw(0.05), search=search)
    r.close()
