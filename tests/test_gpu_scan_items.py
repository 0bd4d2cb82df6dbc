"""Scan work items: lists around the item sizes (64 to 2,048 candidates), few
and many of them, and workspaces with room only for full-size items' descriptors,
against each other (the same scores and ids, bit for bit: an item's size does not
change a candidate's products) and against float64 scores of the records."""

import ctypes as C

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda"


def _index(R, plan, sizes, g):
    sizes = torch.tensor(sizes, dtype=torch.int32, device=DEV)
    padded = (sizes.long() + 15) // 16 * 16
    offsets = torch.cumsum(padded, 0) - padded
    total = int(padded.sum())
    codes = torch.randint(0, 256, (plan.code_bytes(total),), generator=g, device=DEV, dtype=torch.uint8)
    scales = torch.randint(58 << 9, 61 << 9, (total,), generator=g, device=DEV, dtype=torch.int32) | (0x7000 << 16)
    ids = torch.randperm(total, generator=g, device=DEV).to(torch.int32)
    return R.Index(offsets, sizes, ids, codes, scales), total


def _dots(R, plan, index, total, q_rot, bits, D):
    """s^ <q_rot, c^> of every record, float64 (g^ = 1)."""
    cb = synth.codebook(bits).astype(np.float64)
    canon = R.rslm_unpack_codes(plan, index.codes, total).cpu().numpy()
    codes = oracle.unpack_canonical(canon, bits, -(-D // cb.shape[1]))
    chat = torch.from_numpy(cb[codes].reshape(total, -1)[:, :D].copy()).to(DEV)
    u, at = np.unique(index.scales.cpu().numpy() & 0xffff, return_inverse=True)
    sh = torch.from_numpy(np.array([oracle.dec_ue7m9(int(v)) for v in u])[at]).to(DEV)
    return sh * (q_rot.double() @ chat.T)


CASES = [
    # D, bits, list sizes, Q, nprobe: one list a query and every list
    (64, 4, [1], 1, 1),
    (64, 4, [63, 64, 65], 1, 3),
    (96, 2, [127, 128, 129, 0, 640], 2, 5),
    (64, 1, [2047, 2048, 2049], 1, 3),
    (40, 4, [4111, 5, 2050, 70], 9, 4),
    (64, 3, [700] * 40, 3, 13),
    (800, 2, [95] * 60, 17, 6),          # byte table (two workgroups per CU)
    (1200, 3, [250] * 24, 2, 6),         # in passes
    (64, 4, [30] * 700, 40, 18),         # about as many items as workgroups
    (128, 4, [300, 5000] * 30, 64, 20),
]


@pytest.mark.parametrize("D,bits,sizes,Q,nprobe", CASES)
def test_item_sizes(D, bits, sizes, Q, nprobe):
    import paper_2608_30384_amd as R
    from paper_2608_30384_amd import _lib as L
    lib = L.lib()
    g = torch.Generator(device=DEV).manual_seed(D + Q)
    plan = R.Plan(D, bits, passes=1, scale_mode="global")
    index, total = _index(R, plan, sizes, g)
    nlist, k = len(sizes), 20
    q = torch.randn(Q, D, generator=g, device=DEV)
    pid = torch.stack([torch.randperm(nlist, generator=g, device=DEV)[:nprobe] for _ in range(Q)]).to(torch.int32)
    pdot = torch.randn(Q, nprobe, generator=g, device=DEV)
    cs = index.c_struct()
    full = lib.rslm_scan_topk_workspace(plan.handle, C.byref(cs), Q, nprobe, k)
    p = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731

    def scan(nbytes):
        ws = torch.empty(full, dtype=torch.uint8, device=DEV)
        s = torch.full((Q, k), 7.0, device=DEV)
        i = torch.full((Q, k), -7, dtype=torch.int32, device=DEV)
        st = lib.rslm_scan_topk(plan.handle, C.byref(cs), p(q), Q, p(pid), p(pdot), nprobe, k, p(s), p(i),
                                p(ws), nbytes, C.c_void_p(torch.cuda.current_stream().cuda_stream))
        return st, s, i

    st, s, i = scan(full)
    assert st == 0
    lo, hi = 0, full                     # the least workspace that is accepted
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if scan(mid)[0] == 0:
            hi = mid
        else:
            lo = mid
    assert scan(lo)[0] == 4
    st, s2, i2 = scan(hi)
    assert st == 0 and torch.equal(s, s2) and torch.equal(i, i2)
    # against float64: candidates of the probed lists, best scores first.  A score is
    # a float32 sum of D / 32 + 8 roundings of at most ||q|| ||s^ c^||, the query in
    # 22 bits: 1e-5 of the largest leaves room for the sums being larger than it
    dots = _dots(R, plan, index, total, q, bits, D)
    lists = torch.repeat_interleave(torch.arange(nlist, device=DEV), (index.list_sizes.long() + 15) // 16 * 16)
    inside = torch.arange(total, device=DEV) - index.list_offsets[lists] < index.list_sizes[lists]
    for a in range(Q):
        slot = torch.full((nlist,), -1, dtype=torch.long, device=DEV)
        slot[pid[a].long()] = torch.arange(nprobe, device=DEV)
        rec = torch.nonzero(inside & (slot[lists] >= 0))[:, 0]
        sc = pdot[a, slot[lists[rec]]].double() + dots[a, rec]
        n = min(k, len(rec))
        want = torch.sort(sc, descending=True).values[:n]
        tol = 1e-5 * float(sc.abs().max()) + 1e-6
        assert bool(((s[a, :n].double() - want).abs() <= tol).all())
        assert bool((i[a, n:] == -1).all()) and bool(torch.isneginf(s[a, n:]).all())
        by_id = {int(v): float(w) for v, w in zip(index.ids[rec].tolist(), sc.tolist())}
        assert all(abs(by_id[int(v)] - float(w)) <= tol for v, w in zip(i[a, :n].tolist(), s[a, :n].tolist()))
