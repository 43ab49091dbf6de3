"""Where the workgroups of a thresholded layer write their parts of the message: single workgroups, their edges, and more of them
than a workgroup's threads take the counts of in one step (16 x 256)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[1, 16_383, 16_384, 16_385], [3 * 16_384 + 1, 16 * 16_384], [4098 * 32_768 + 5]])
def test_reused_threshold(sizes):
    import torch
    import paper_1808_04357_amd as rgc
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sizes[0])
    V = [torch.empty(n, device="cuda").normal_(0.0, 1.0, generator=gen) for n in sizes]
    G = [torch.zeros(n, device="cuda") for n in sizes]
    want = [v.clone() for v in V]
    ks = [max(1, n // 500) for n in sizes]
    thr = torch.full((len(sizes),), 3.0, device="cuda")            # 0.27 % of normal values lie above it
    nnz = torch.full((len(sizes),), -1, dtype=torch.int32, device="cuda")
    idx = [torch.full((2 * k,), -1, dtype=torch.int32, device="cuda") for k in ks]
    val = [torch.full((2 * k,), float("nan"), device="cuda") for k in ks]
    cnt = torch.full((len(sizes),), -1, dtype=torch.int32, device="cuda")
    ctx = rgc.Context(sum(sizes), len(sizes))
    layers = rgc.LayerList(G, V, ks, idx, val, cnt)
    for t in range(2):                                             # the second call finds nothing new above the threshold
        rgc.rgc_compress_layers_threshold(ctx, layers, 0.0, thr, nnz, 0)
        torch.cuda.synchronize()
        for l, k in enumerate(ks):
            at = torch.nonzero(want[l].abs() > 3.0).flatten()
            sent = at[:2 * k]
            assert int(nnz[l]) == at.numel() and int(cnt[l]) == sent.numel()
            assert torch.equal(idx[l][:sent.numel()].long(), sent)
            assert torch.equal(val[l][:sent.numel()], want[l][sent])
            want[l][sent] = 0.0
            assert torch.equal(V[l], want[l])
    ctx.close()
