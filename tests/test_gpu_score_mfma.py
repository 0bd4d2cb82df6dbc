"""OneToMany scoring on the matrix cores at the edges of its shapes (chunk
counts, partial last chunks, ragged last tiles, one to five queries, records
at the very end of the pool) against float64 scores of the same records.
The bound is that of a float32 dot product: D / 32 + 8 roundings of partial
sums no larger than ||q|| ||C[code]||, times the two scales."""

import ctypes as C

import numpy as np
import pytest

import oracle
import synth
from tests import helpers as H

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda"


def _records(R, D, bits, mode, n, seed):
    plan = R.Plan(D, bits, passes=1, scale_mode=mode)
    rng = np.random.default_rng(seed)
    C = synth.codebook(bits).astype(np.float64)
    codes = rng.integers(0, C.shape[0], (n, -(-D // C.shape[1])))
    su = rng.integers((58 << 9), (61 << 9), n)
    gu = rng.integers((6 << 12), (8 << 12), n) if mode == "global" else np.full(n, 0x7000)
    recs = oracle.pack_records(codes, su, gu, bits, mode)
    sh, gh = H.dec_scales(su.astype(np.uint32) | (gu.astype(np.uint32) << 16))
    chat = C[codes].reshape(n, -1)[:, :D]
    return plan, torch.from_numpy(np.ascontiguousarray(recs)).to(DEV), sh * gh, chat


@pytest.mark.parametrize("D,bits,mode,Q", [
    (1, 4, "local", 1), (31, 4, "global", 4), (32, 3, "local", 5), (33, 2, "global", 1), (64, 1, "local", 3),
    (97, 4, "global", 2), (130, 1, "global", 1), (200, 3, "global", 1), (255, 4, "local", 1),
    (257, 2, "local", 4), (300, 3, "local", 1), (511, 4, "global", 1), (513, 4, "local", 1),
    (700, 1, "local", 1), (768, 3, "global", 5), (777, 4, "global", 1), (945, 2, "global", 1),
    (1023, 1, "global", 2), (1024, 4, "local", 1), (1024, 3, "local", 1)])
def test_against_float64(D, bits, mode, Q):
    import paper_2608_30384_amd as R
    n = 4099
    plan, recs, scale, chat = _records(R, D, bits, mode, n, D)
    q = np.random.default_rng(D + 1).standard_normal((Q, D)).astype(np.float32)
    q[0] *= 1e-3
    ref = (q.astype(np.float64) @ chat.T) * scale
    bound = (D / 32 + 8) * 2.0 ** -24 * np.linalg.norm(q, axis=1)[:, None] * np.linalg.norm(chat, axis=1) * scale
    got = R.rslm_score(plan, recs, torch.from_numpy(q).to(DEV)).cpu().numpy()
    assert np.all(np.abs(got - ref) <= bound)
    ids = np.random.default_rng(D + 2).integers(0, n, 5000)
    ids[:2], ids[2], ids[-1] = [-1, n], n - 1, n - 1
    got = R.rslm_score(plan, recs, torch.from_numpy(q).to(DEV),
                       ids=torch.from_numpy(ids).to(DEV)).cpu().numpy()
    assert np.all(np.isneginf(got[:, :2]))
    assert np.all(np.abs(got[:, 2:] - ref[:, ids[2:]]) <= bound[:, ids[2:]])


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
def test_special_queries(bits):
    """Infinite and NaN coordinates as in a plain sum (no centroid value is 0
    here); a query of zeros scores 0; another query of the group is untouched."""
    import paper_2608_30384_amd as R
    D, n = 96, 5000
    plan, recs, scale, chat = _records(R, D, bits, "local", n, 5)
    q = np.random.default_rng(6).standard_normal((4, D)).astype(np.float32)
    q[1] = 0.0
    q[2, 7] = np.inf
    q[3, 9] = np.nan
    got = R.rslm_score(plan, recs, torch.from_numpy(q).to(DEV)).cpu().numpy()
    ref = (q[0].astype(np.float64) @ chat.T) * scale
    assert np.all(np.abs(got[0] - ref) <= 1e-5 * np.linalg.norm(q[0]) * np.linalg.norm(chat, axis=1) * scale)
    assert not got[1].any()
    sign = np.sign(chat[:, 7])
    assert np.all(got[2][sign != 0] == np.inf * sign[sign != 0])
    assert np.isnan(got[3]).all()


@pytest.mark.parametrize("D,bits,mode", [(64, 4, "global"), (300, 3, "local"), (1024, 1, "global")])
@pytest.mark.parametrize("Q", [1, 5])
def test_empty_pool(D, bits, mode, Q):
    """No record to read: every id is outside the pool and scores -inf (through the C
    entry point, as torch gives an empty tensor a null pointer)."""
    import paper_2608_30384_amd as R
    from paper_2608_30384_amd import _lib as L
    plan = R.Plan(D, bits, passes=1, scale_mode=mode)
    n = 8192
    pool = torch.zeros(16, dtype=torch.uint8, device=DEV)
    ids = torch.randint(-3, 4, (n,), device=DEV)
    q = torch.randn(Q, D, device=DEV)
    out = torch.full((Q, n), 7.0, device=DEV)
    p = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
    assert L.lib().rslm_score(plan.handle, p(pool), 0, p(ids), n, p(q), Q, p(out),
                              C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    assert bool(torch.isneginf(out).all())
