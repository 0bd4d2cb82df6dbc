"""Centre updates with few centres (shared runs, counts in LDS) against float64
means: at the sizes where the number of shares and the counting change, with
empty centres, assignments out of range, and workspaces without room for the
partial sums or 4 bytes past their alignment.  A mean is rounded to float32 once: 2^-24 relative, and the
float64 sums add less than n 2^-53."""

import ctypes as C

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("n,dim,nlist", [
    (127, 5, 1), (128, 300, 1), (70001, 3, 1), (4096, 64, 16), (40000, 257, 16), (100000, 1, 7),
    (32768, 96, 16), (32767, 96, 16), (300000, 20, 140), (131072, 31, 1024), (9000, 40, 4097)])
@pytest.mark.parametrize("room,shift", [(True, 0), (False, 0), (True, 4)])
def test_update_of_few_centres(n, dim, nlist, room, shift):
    from paper_2608_30384_amd import _lib as L
    g = torch.Generator(device=DEV).manual_seed(n + dim)
    x = torch.randn(n, dim, generator=g, device=DEV) + 0.5
    a = torch.randint(0, nlist, (n,), generator=g, device=DEV, dtype=torch.int32)
    if nlist > 3:
        a[a == 2] = 3                       # an empty centre
    a[::97] = -1
    a[5::1013] = nlist                      # out of range
    c = torch.full((nlist, dim), 7.0, device=DEV)
    align = lambda b: (b + 255) // 256 * 256  # noqa: E731
    least = 2 * align(nlist * 4) + align((nlist + 1) * 4) + align(n * 4)
    full = L.lib().ivf_kmeans_update_workspace(n, nlist)
    assert full >= least
    ws = torch.empty((full if room else least) + shift, dtype=torch.uint8, device=DEV)[shift:]
    p = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
    args = (p(x), n, dim, p(a), nlist, p(c), p(ws))
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert L.lib().ivf_kmeans_update(*args, least - 256, s) == 4   # too small: refused
    assert L.lib().ivf_kmeans_update(*args, ws.numel(), s) == 0
    ok = (a >= 0) & (a < nlist)
    want = torch.zeros(nlist, dim, dtype=torch.float64, device=DEV).index_add_(
        0, a[ok].long(), x[ok].double())
    cnt = torch.bincount(a[ok].long(), minlength=nlist)[:, None]
    want = torch.where(cnt > 0, want / cnt.clamp(min=1), torch.full_like(want, 7.0))
    size = x.abs().max().double()
    assert bool(((c.double() - want).abs() <= 2.0 ** -24 * want.abs() + n * 2.0 ** -53 * size).all())
