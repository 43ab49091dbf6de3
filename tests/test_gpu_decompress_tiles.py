"""GPU parity of the decompression around the sizes of its tiles and the densities that choose them (bit equality)."""
import numpy as np
import pytest

from test_gpu_decompress import compare, gpu_decompress, oracle_all, random_messages

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rgc():
    import paper_1808_04357_amd as m
    return m


# entries of a worker in 8192 positions: 2048 above 64 and 22, 4096 above 11 and 13 to 17 (and in small calls of up to 64 workers), else 8192
@pytest.mark.parametrize("add", [False, True])
@pytest.mark.parametrize("per_8192", [5, 12, 20, 40, 90])
@pytest.mark.parametrize("workers", [1, 3, 64, 65, 128, 130])
def test_tile_edges(rgc, oracle, workers, per_8192, add):
    """Layers that end at, just before and just behind a tile of each size, with ends of 1 to 3 elements behind the last
    whole 16 bytes, on unaligned buffers; the same from tiles of 8192 positions in a call that is not small."""
    g = np.random.default_rng(1000 * workers + per_8192)
    sizes = [1, 3, 2047, 2048, 2049, 4095, 4098, 8189, 8192, 8195, 2 * 8192 + 1, 5 * 2048 - 2]
    counts = [max(1, n * per_8192 // 8192) for n in sizes]
    hot = [g.choice(n, size=max(1, n // 300), replace=False) for n in sizes]
    idx, val = random_messages(g, sizes, workers, counts, hot)
    init = [g.standard_normal(n).astype(np.float32) for n in sizes] if add else None
    ctx = rgc.Context(sum(sizes), len(sizes))
    got = gpu_decompress(rgc, ctx, idx, val, sizes, 0.7, init, misalign=per_8192 % 4)
    compare("%d workers, %d" % (workers, per_8192), got, oracle_all(oracle, idx, val, sizes, 0.7, init))
    ctx.close()


@pytest.mark.parametrize("workers", [2, 7])
def test_large_tiles_for_few_workers(rgc, oracle, workers):
    """From 32 Mi elements on the messages of few workers are added in tiles of 8192 positions, too."""
    g = np.random.default_rng(workers)
    sizes = [(32 << 20) + 8189, 8193]
    pos = np.sort(g.choice(sizes[0], size=30_000, replace=False)).astype(np.int32)
    idx = [[pos[g.random(pos.size) < 0.8], np.arange(w, 8193, 700, dtype=np.int32)] for w in range(workers)]
    val = [[g.standard_normal(i.size).astype(np.float32) for i in row] for row in idx]
    ctx = rgc.Context(sum(sizes), len(sizes))
    got = gpu_decompress(rgc, ctx, idx, val, sizes, 1.0 / workers, None, misalign=1)
    compare("%d workers" % workers, got, oracle_all(oracle, idx, val, sizes, 1.0 / workers, None))
    ctx.close()


# entries of all workers in 8192 positions: (3, 6) .. (128, 105) are paced with 1, 2, 4, 1 and 2 stores at once, (1, 12) and (2, 30) with 1 in
# tiles of 4096; the others are not, nor is any call that adds
@pytest.mark.parametrize("mode", ["overwrite", "add", "one value"])
@pytest.mark.parametrize("workers,in_8192", [(1, 12), (2, 30), (3, 6), (16, 20), (64, 45), (65, 60), (128, 105), (3, 100), (7, 2), (64, 200), (128, 200)])
def test_few_entries_in_large_buffers(rgc, oracle, workers, in_8192, mode):
    """The tiles of calls on 48 Mi elements and more; in the small layers a worker has more entries than its window holds, and
    more positions collide than there are rows."""
    import torch
    g = np.random.default_rng(100 * workers + in_8192)
    sizes = [(48 << 20) + 8189, 8189, 8193, 3 * 8192 + 2, 5]
    count = in_8192 * 6144 // workers
    shared = [g.integers(0, n, size=2 * count if l == 0 else n // 70 + 1) for l, n in enumerate(sizes)]
    idx = [[np.unique(np.concatenate([g.choice(s, size=s.size // 4 + 1), g.integers(0, n, size=count // 2 if l == 0 else n // 250 + 1)])).astype(np.int32)
            for l, (n, s) in enumerate(zip(sizes, shared))] for _ in range(workers)]
    one = mode == "one value"
    val = [[g.standard_normal(1 if one else i.size).astype(np.float32) for i in row] for row in idx]
    assert max(i.size for row in idx for i in row[1:4]) > 50
    dev = torch.device("cuda:0")
    init = [g.standard_normal(n).astype(np.float32) for n in sizes] if mode == "add" else None
    dense = [torch.full((n + 1,), float("nan"), device=dev)[1:] for n in sizes]
    if init is not None:
        for d, i in zip(dense, init):
            d.copy_(torch.from_numpy(i))
    up = lambda rows: [[torch.from_numpy(a).to(dev) for a in row] for row in rows]
    ctx = rgc.Context(sum(sizes), len(sizes))
    flags = (rgc.RGC_ADD_TO_DST if init is not None else rgc.RGC_OVERWRITE) | (rgc.RGC_ONE_VALUE if one else 0) | rgc.RGC_VALIDATE
    rgc.rgc_decompress_accumulate(ctx, rgc.MessageList(up(idx), up(val), dense), 0.7, flags, torch.cuda.current_stream())
    torch.cuda.synchronize()
    if one:
        val = [[v.repeat(i.size) for v, i in zip(*rows)] for rows in zip(val, idx)]
    compare("%d workers, %d, %s" % (workers, in_8192, mode), [d.cpu().numpy() for d in dense], oracle_all(oracle, idx, val, sizes, 0.7, init))
    ctx.close()
