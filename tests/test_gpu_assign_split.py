"""Assignment on split float16 (large ``ivf_assign_probe`` L2 calls) at the edges
of its tiles -- 256 rows, 256 centres, slabs of 32 coordinates, shares of the
centres -- against float64: the chosen centre is within the bound of the
nearest, and the distance within it of that centre's.  The bound is that of a
float32 evaluation of ||x||^2 + (||c||^2 - 2 <x, c>): each of the D / 32
additions and the few others rounds values of at most (||x|| + ||c||)^2 by 2^-24.
The calls that run on split float16 meet more: the nearest centre in float64,
whatever the spread of the values, and the same results with any workspace.
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
    (1500, 1447, 513), (70000, 65, 16), (3000, 1, 400),
    # (on the float32 kernels: those above with few centres or coordinates)
    (128, 16, 4096), (255, 200, 512), (256, 96, 1025), (257, 36, 4097), (1000, 192, 513), (700, 230, 1),
    (129, 67, 400), (2000, 33, 1100), (300, 1021, 257), (4573, 230, 21), (127, 230, 300),
    (131072, 128, 129), (65537, 131, 16), (65536, 97, 131)])
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


@pytest.mark.parametrize("dim", [40, 84, 85])
def test_ties_take_the_lowest_id(R, dim):
    """Integer-valued vectors (every product exact): equal centres in one lane's
    run, in two lanes', in two wavefronts' and in two tiles and shares."""
    g = torch.Generator(device=DEV).manual_seed(1)
    c = torch.randint(-8, 9, (1200, dim), generator=g, device=DEV).float()
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


@pytest.mark.parametrize("dim", [64, 67, 164])
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
    c = torch.randn(1100, 96, device=DEV)
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


# ---- the centre that is nearest in float64, whatever the values' spread
def _nearest(x, c, ids, dist):
    """The chosen centre is the nearest up to float64 roundings, and the distance
    is that of float64 rounded once (2^-24, and 2^-50 of the values summed)."""
    x64, c64 = x.double(), c.double()
    r = (c64 * c64).sum(1) - 2 * x64 @ c64.T
    size = (x64.abs() @ c64.abs().T).max(1).values + (c64 * c64).sum(1).max()
    got = r.gather(1, ids.long()[:, None])[:, 0]
    assert bool((got - r.min(1).values <= 2.0 ** -44 * size).all())
    own = ((x64 - c64[ids.long()]) ** 2).sum(1)
    assert bool(((dist.double() - own).abs() <= 2.0 ** -23 * own + 1e-44).all())


@pytest.mark.parametrize("dim", [16, 17, 32, 48, 64, 67, 100, 1447])
@pytest.mark.parametrize("kind", ["plain", "spike", "small", "large", "ties", "offset"])
def test_nearest_in_float64(R, dim, kind):
    g = torch.Generator(device=DEV).manual_seed(dim)
    # (sizes that run on split float16; with 70,000 listed rows the centres are not shared out)
    n, nlist = 70000 if kind == "ties" and dim == 17 else 1500, max(600, 4200 if dim < 50 else 1600 if dim < 101 else 0)
    c = torch.randn(nlist, dim, generator=g, device=DEV)
    x = c[torch.randint(0, nlist, (n,), generator=g, device=DEV)] + \
        0.8 * torch.randn(n, dim, generator=g, device=DEV)
    if kind == "spike":      # one coordinate far above the rest, where the centres are 0
        c[:, 2] = 0.0
        x[:, 2] = 10.0 ** (2 + torch.arange(n, device=DEV) % 10).float()
    elif kind == "small":    # the product of two scales is below the smallest float32
        x, c = x * 1e-19, c * 1e-19
    elif kind == "large":
        x, c = x * 1e15, c * 1e15
    elif kind == "ties":     # each centre and copies of it one rounding away
        c[nlist // 2:] = c[:nlist // 2] * (1 + 2.0 ** -23)
        c[nlist // 3: nlist // 2] = c[:nlist // 2 - nlist // 3]
    elif kind == "offset":
        x, c = x + 300.0, c + 300.0
    ids, dist = R.ivf_assign_probe(x, c, 1, R.IVF_ASSIGN_L2)
    _nearest(x, c, ids, dist)
    if kind == "ties":       # exact copies: the lower id
        copies = torch.arange(nlist // 3, nlist // 2, device=DEV, dtype=torch.int32)
        assert not bool(torch.isin(ids, copies).any())


@pytest.mark.parametrize("n,dim,nlist", [(300, 768, 24576), (40000, 100, 3000), (5000, 230, 40)])
def test_workspace_and_pieces_do_not_change_results(R, n, dim, nlist):
    """The queried workspace, smaller and larger ones, one sized for a larger n and the
    allocation-free entry point: the same ids and distances."""
    from paper_2608_30384_amd import _lib as L
    g = torch.Generator(device=DEV).manual_seed(n)
    c = torch.randn(nlist, dim, generator=g, device=DEV)
    x = c[torch.randint(0, nlist, (n,), generator=g, device=DEV)] + torch.randn(n, dim, generator=g, device=DEV)
    want = R.ivf_assign_probe(x, c, 1, R.IVF_ASSIGN_L2)
    _nearest(x[:300], c, want[0][:300], want[1][:300])
    lib = L.lib()
    p = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    full = lib.ivf_assign_probe_workspace(n, dim, nlist, 1, R.IVF_ASSIGN_L2)
    assert full <= lib.ivf_assign_probe_noalloc_limit()
    sizes = [full, 2 * full, lib.ivf_assign_probe_workspace(50 * n, dim, nlist, 1, R.IVF_ASSIGN_L2)]
    if n > 4096:             # (calls of fewer rows are not cut for a smaller workspace)
        sizes += [full - 256] + ([full * 3 // 4] if n > 16384 else [])
    for size in sizes:
        ids = torch.full((n,), -7, dtype=torch.int32, device=DEV)
        dist = torch.full((n,), 7.0, device=DEV)
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        assert lib.ivf_assign_probe(p(x), n, dim, p(c), nlist, 1, R.IVF_ASSIGN_L2, p(ids), p(dist), p(ws),
                                    size, stream) == 0
        assert torch.equal(ids, want[0]) and torch.equal(dist, want[1])
    ids, dist = torch.full_like(ids, -7), torch.full_like(dist, 7.0)
    assert lib.ivf_assign_probe_noalloc(p(x), n, dim, p(c), nlist, 1, R.IVF_ASSIGN_L2, p(ids), p(dist), stream) == 0
    assert torch.equal(ids, want[0]) and torch.equal(dist, want[1])
    ids = torch.full_like(ids, -7)   # without distances
    ws = torch.empty(full, dtype=torch.uint8, device=DEV)
    assert lib.ivf_assign_probe(p(x), n, dim, p(c), nlist, 1, R.IVF_ASSIGN_L2, p(ids), C.c_void_p(0), p(ws),
                                full, stream) == 0
    assert torch.equal(ids, want[0])


@pytest.mark.parametrize("n", [128, 256, 257, 4100])
@pytest.mark.parametrize("dim", [96, 230, 1100])
def test_rows_settled_in_float64(R, n, dim):
    """Every row listed (each centre and a copy one rounding away): numbers of rows
    around where the float64 kernel changes its tile."""
    g = torch.Generator(device=DEV).manual_seed(n + dim)
    nlist = 1101
    c = torch.randn(nlist, dim, generator=g, device=DEV)
    c[nlist // 2:2 * (nlist // 2)] = c[:nlist // 2] * (1 + 2.0 ** -23)
    x = c[torch.randint(0, nlist, (n,), generator=g, device=DEV)] + torch.randn(n, dim, generator=g, device=DEV)
    ids, dist = R.ivf_assign_probe(x, c, 1, R.IVF_ASSIGN_L2)
    _nearest(x, c, ids, dist)
