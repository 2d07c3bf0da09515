"""The early prediction in one launch at the edges of its blocks of columns, runs of rows and lists, against 64 bits."""
import numpy as np
import pytest
import torch

from paper_2307_05908_amd import binding

pytestmark = pytest.mark.gpu


def inputs(K, V, dtype, seed, offset=0):
    gen = torch.Generator().manual_seed(seed)
    def place(t):                                   # `offset` elements behind a 16-byte boundary
        buf = torch.zeros(len(t) + 8, dtype=t.dtype).cuda()
        buf[offset:offset + len(t)] = t.cuda()
        return buf[offset:offset + len(t)]
    h = (1.5 * torch.randn(K, generator=gen) + 0.3).cuda()
    g = place((1 + 0.1 * torch.randn(K, generator=gen)).to(dtype))
    b = place((0.1 * torch.randn(K, generator=gen)).to(dtype))
    return h, g, b, (0.05 * torch.randn(V, K, generator=gen)).to(dtype).cuda()


def check(fn, h, g, b, head, k, norm):
    K = len(h)
    ids, vals, z = fn(h, g, b if norm == 0 else None, head, k, norm, 1e-5, want_logits=True)
    torch.cuda.synchronize()
    z, ids = z.cpu().numpy(), ids.cpu().numpy()
    x = h.double()
    x = x - x.mean() if norm == 0 else x
    x = x / torch.sqrt((x * x).mean() + 1e-5) * g.double()
    x = x + b.double() if norm == 0 else x
    w = head.double()
    ref, size = (w @ x).cpu().numpy(), (w.abs() @ x.abs()).cpu().numpy()
    # a lane adds at most 80 products in turn, then six levels of lanes; the row's own rounding: statistics, three products and a sum
    assert (np.abs(z - ref) <= size * (80 + 6 + 16) * 2.0 ** -24).all()
    order = np.lexsort((np.arange(len(z)), -z.astype(np.float64)))[:k]
    np.testing.assert_array_equal(ids, order)
    np.testing.assert_array_equal(vals.cpu().numpy(), z[order])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("norm", [0, 1])
@pytest.mark.parametrize("K", [8, 248, 256, 264, 504, 512, 520, 1016, 1032, 1536, 1544, 2048, 2056, 2560, 2568, 3080, 4096, 4104, 5112, 5120, 5128])
def test_columns(K, norm, dtype):
    V = 613
    h, g, b, head = inputs(K, V, dtype, K)
    check(binding.ppd_early_topk_noalloc, h, g, b, head, 5, norm)
    h, g, b, head = inputs(K, V, dtype, K, offset=1)          # gains and biases that no 16-byte load may take
    check(binding.ppd_early_topk, h, g, b, head, 8, norm)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V", [1, 3, 15, 16, 17, 63, 1000, 4095, 4096, 4097, 16384, 65535, 65536])
def test_rows(V, dtype):
    for K, k in ((64, 8), (768, 1)):
        h, g, b, head = inputs(K, V, dtype, V)
        check(binding.ppd_early_topk_noalloc, h, g, b, head, min(k, V), 1)


@pytest.mark.parametrize("V", [65537, 131072, 131073, 300000])       # up to and beyond 512 lists
def test_more_lists(V):
    h, g, b, head = inputs(64, V, torch.bfloat16, V)
    head[V // 2:] = head[:V - V // 2].clone()                        # every logit twice
    check(binding.ppd_early_topk, h, g, b, head, 8, 0)


def test_logits_that_are_no_numbers_are_no_candidates():
    h, g, b, head = inputs(256, 2000, torch.float32, 5)
    head[7] = float("nan")
    head[1234] = float("nan")
    ids, vals, z = binding.ppd_early_topk(h, g, None, head, 8, 1, 1e-5, want_logits=True)
    z = z.cpu().numpy()
    assert np.isnan(z[[7, 1234]]).all() and np.isnan(z).sum() == 2
    np.testing.assert_array_equal(ids.cpu().numpy(), np.argsort(np.where(np.isnan(z), np.inf, -z), kind="stable")[:8])
    head[:] = float("nan")
    ids, _, _ = binding.ppd_early_topk(h, g, None, head, 3, 1, 1e-5)
    np.testing.assert_array_equal(ids.cpu().numpy(), [0x7fffffff] * 3)


def test_replayed_calls_of_several_sizes():
    """Captured, with calls of other grids and the program's own work between the replays."""
    cases = [inputs(K, V, torch.bfloat16, K + V) for K, V in ((512, 5000), (64, 300), (1024, 40000))]
    fn = binding.ppd_early_topk_noalloc
    refs = [[t.cpu() for t in fn(h, g, b, head, 8, 0, 1e-5, want_logits=True)] for h, g, b, head in cases]
    stream = torch.cuda.Stream()
    graphs = []
    for h, g, b, head in cases:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            out = fn(h, g, b, head, 8, 0, 1e-5, want_logits=True)
        graphs.append((graph, out))
    for i in (0, 1, 2, 1, 1, 0, 2, 2, 0):
        for t in graphs[i][1]:
            t.zero_()
        graphs[i][0].replay()
        torch.cuda.synchronize()
        for t, r in zip(graphs[i][1], refs[i]):
            assert torch.equal(t.cpu(), r)
        fn(*cases[(i + 1) % 3], 2, 0, 1e-5)
