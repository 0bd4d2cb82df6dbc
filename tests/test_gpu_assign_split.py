"""Assignment on split float16 (large ``ivf_assign_probe`` L2 calls) at the edges
of its tiles -- 256 rows, 256 centres, slabs of 32 coordinates, shares of the
centres -- against float64: the chosen centre is within the bound of the
nearest, and the distance within it of that centre's.  The bound is that of a
float32 evaluation of ||x||^2 + (||c||^2 - 2 <x, c>): each of the D / 32
additions and the few others rounds values of at most (||x|| + ||c||)^2 by 2^-24.
"""

import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.fixture(scope="module")
def R():
    import paper_2608_30384_amd as R
    return R


def _check(x, c, ids, dist):
    x64, c64 = x.double(), c.double()
    d = (x64 * x64).sum(1)[:, None] - 2 * x64 @ c64.T + (c64 * c64).sum(1)
    got = d.gather(1, ids.long()[:, None])[:, 0]
    size = (x64.norm(dim=1) + c64.norm(dim=1).max()) ** 2
    bound = (x.shape[1] / 32 + 8) * 2.0 ** -24 * size
    assert bool((got - d.min(1).values <= 2 * bound).all())
    assert bool(((dist.double() - got).abs() <= bound).all())


@pytest.mark.parametrize("n,dim,nlist", [
    (128, 32, 129), (255, 64, 256), (256, 96, 257), (257, 36, 511), (1000, 100, 1000),
    (300, 768, 4096), (513, 4, 300), (2000, 33, 40), (700, 31, 129), (4573, 230, 21),
    (1500, 1447, 513), (70000, 65, 16), (3000, 1, 400)])
def test_against_float64(R, n, dim, nlist):
    g = torch.Generator(device=DEV).manual_seed(n + dim)
    c = torch.randn(nlist, dim, generator=g, device=DEV) * 0.7 + 0.3
    x = c[torch.randint(0, nlist, (n,), generator=g, device=DEV)] + \
        0.8 * torch.randn(n, dim, generator=g, device=DEV)
    x[0] = 0.0
    x[1] *= 1e-20          # scales far from 1, per row
    x[2] *= 1e6
    c[nlist // 2] *= 1e-12
    ids, dist = R.ivf_assign_probe(x, c, 1, R.IVF_ASSIGN_L2)
    _check(x, c, ids, dist)


def test_ties_take_the_lowest_id(R):
    """Integer-valued vectors (every product exact): equal centres in one lane's
    run, in two lanes', in two wavefronts' and in two tiles and shares."""
    g = torch.Generator(device=DEV).manual_seed(1)
    c = torch.randint(-8, 9, (1200, 40), generator=g, device=DEV).float()
    for a, b in ((5, 6), (9, 700), (40, 200), (300, 301), (511, 1199), (0, 1023)):
        c[b] = c[a]
    x = c[torch.arange(1200, device=DEV)].repeat(2, 1)
    ids, dist = R.ivf_assign_probe(x, c, 1, R.IVF_ASSIGN_L2)
    first = torch.tensor([int((c == row).all(1).nonzero()[0]) for row in c], device=DEV)
    assert torch.equal(ids.long(), first.repeat(2))
    assert bool((dist == 0).all())


def _float32_path(R, x, c):
    """The same call with a workspace that has room for the norms only."""
    from paper_2608_30384_amd import _lib as L
    n, dim = x.shape
    nlist = c.shape[0]
    ids = torch.empty(n, dtype=torch.int32, device=DEV)
    dist = torch.empty(n, device=DEV)
    ws = torch.empty((nlist * 4 + 255) // 256 * 256, dtype=torch.uint8, device=DEV)
    p = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
    st = L.lib().ivf_assign_probe(p(x), n, dim, p(c), nlist, 1, R.IVF_ASSIGN_L2, p(ids), p(dist), p(ws),
                                  ws.numel(), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    return ids, dist


@pytest.mark.parametrize("dim", [64, 67])
def test_special_values_and_small_workspace(R, dim):
    """Infinities and NaN give what the float32 kernels give, which also run
    (and agree) when the workspace holds no more than their scratch."""
    g = torch.Generator(device=DEV).manual_seed(dim)
    c = torch.randn(600, dim, generator=g, device=DEV)
    x = torch.randn(400, dim, generator=g, device=DEV)
    ids, dist = R.ivf_assign_probe(x, c, 1, R.IVF_ASSIGN_L2)
    ids32, dist32 = _float32_path(R, x, c)
    assert float((ids == ids32).float().mean()) > 0.99
    assert bool(((dist - dist32).abs() <= 1e-4 * dist32.abs()).all())
    x[7, 3] = float("nan")
    x[8, 5] = float("inf")
    x[9, 6] = float("-inf")
    x[10, 0], x[10, 1] = float("inf"), float("nan")
    x[11, 2] = 3e38
    c[12, 4] = float("inf")
    c[13, 4] = float("nan")
    ids, dist = R.ivf_assign_probe(x, c, 1, R.IVF_ASSIGN_L2)
    ids32, dist32 = _float32_path(R, x, c)
    rows = [7, 8, 9, 10]
    assert ids[rows].tolist() == ids32[rows].tolist()
    assert torch.equal(torch.isnan(dist[rows]), torch.isnan(dist32[rows]))
    assert not bool(((ids == 12) | (ids == 13)).any())


def test_replays_in_a_graph(R):
    """Captured and replayed with new inputs: every replay as the eager call."""
    c = torch.randn(500, 96, device=DEV)
    x = torch.randn(900, 96, device=DEV)
    ids = torch.empty(900, dtype=torch.int32, device=DEV)
    dist = torch.empty(900, device=DEV)
    run = lambda: R.ivf_assign_probe(x, c, 1, R.IVF_ASSIGN_L2, out_ids=ids, out_scores=dist)  # noqa: E731
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        run()
    for k in range(4):
        x.copy_(torch.randn(900, 96, device=DEV))
        graph.replay()
        torch.cuda.synchronize()
        got = ids.clone(), dist.clone()
        want = R.ivf_assign_probe(x, c, 1, R.IVF_ASSIGN_L2)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
