"""Encoder and decoder on 16-lane rows at the sizes where they change shape:
the smallest and largest dimension of every (rows per vector, blocks per row)
arrangement, with and without an overlapping block, tails from 1 to 127
coordinates, every bit width and second stage, and record counts that leave
rows of the last wavefront without a vector.  Inputs, oracle and tolerances
are those of the parity tests of the same entry points."""

import numpy as np
import pytest

import oracle
import synth
from tests import helpers as H
from tests import test_gpu_parity as parity
from tests import test_gpu_records as records
from tests import test_gpu_rescore_rslm as rescore

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda"
R = parity.R

# (D, bits, passes): block counts 1 (128), 2, 3, 4, 5, 6, 7, 8, 9, 12, 13, 16,
# 17, 20, 21, 24, 25, 28, 29, 32.
DIMS = [(128, 3, 2), (129, 4, 1), (255, 1, 2), (256, 2, 2), (257, 2, 2), (300, 1, 2), (384, 4, 2),
        (384, 2, 1), (385, 4, 2), (386, 4, 2), (512, 3, 2), (513, 2, 2), (640, 1, 2), (700, 3, 2),
        (769, 4, 2), (1000, 2, 2), (1024, 1, 1), (1025, 4, 2), (1500, 3, 2), (1537, 1, 2),
        (2047, 2, 2), (2049, 2, 2), (2560, 4, 2), (2561, 1, 2), (3000, 4, 2), (3073, 3, 2),
        (3584, 2, 2), (3585, 4, 0), (4096, 4, 2)]


@pytest.mark.parametrize("D,bits,passes", DIMS)
def test_encode(R, D, bits, passes):
    parity.test_encode_parity(R, D, bits, passes, "global" if D % 2 else "local")


@pytest.mark.parametrize("D,bits,passes", DIMS)
def test_decode(R, D, bits, passes):
    records.test_decode_parity(R, D, bits, passes, "local" if D % 2 else "global", bits == 4 and D % 3 == 0)


@pytest.mark.parametrize("D,bits,passes,mode2,n", [
    (129, 4, 1, "global", 37), (255, 2, 2, "local", 41), (300, 1, 2, "global", 50),
    (384, 4, 2, "global", 35), (384, 1, 2, "local", 18),
    (385, 3, 2, "global", 33), (640, 4, 2, "local", 30), (1025, 2, 2, "global", 27),
    (1537, 4, 2, "global", 21), (2561, 3, 2, "global", 18), (3585, 4, 2, "global", 19),
    (4096, 1, 2, "local", 18)])
def test_encode_two_stage(R, D, bits, passes, mode2, n):
    rescore.test_encode_two_stage_parity(R, D, bits, passes, 2, mode2, n)


@pytest.mark.parametrize("D,passes,n,lite", [(129, 1, 61, False), (255, 2, 77, True), (300, 2, 90, False),
                                             (384, 2, 49, False), (384, 2, 83, True),
                                             (700, 2, 66, True), (1025, 2, 70, False),
                                             (2049, 2, 75, True), (3001, 2, 60, False),
                                             (4096, 2, 51, False)])
def test_encode_sq8(R, D, passes, n, lite):
    rescore.test_encode_sq8_parity(R, D, passes, n, lite)


@pytest.mark.parametrize("D", [131, 300, 384, 768, 2049])
def test_rows_at_any_alignment(R, D):
    """Rows of x, the centres and the outputs that start 4 bytes past a 16-byte
    boundary (1 byte for codes and codes2), records in any order with unused ones
    among them: the same bytes as aligned arrays in row order; and the same
    vectors decoded from codes at any byte."""
    n, nlist, plan = 53, 4, None
    rng = np.random.default_rng(D)
    x = synth.aniso(n, D, seed=D)
    cen = x[rng.choice(n, nlist, replace=False)] * 0.9
    assign, _ = oracle.assign_l2(x, cen)
    plan = R.Plan(D, 4, passes=2)

    def off(a, k=1):
        t = torch.zeros(a.size + k, dtype=torch.from_numpy(a).dtype, device=DEV)[k:].view(a.shape)
        return t.copy_(torch.from_numpy(np.ascontiguousarray(a)))

    def encode(xt, ct, crot, src, lists, lo, hi, codes2, shift=0):
        m = lists.numel()
        codes = torch.zeros(plan.code_bytes(m) + shift, dtype=torch.uint8, device=DEV)[shift:]
        scales = torch.zeros(m, dtype=torch.int32, device=DEV)
        R.rslm_encode_sq8(plan, xt, codes, scales, lo, hi, codes2, n_records=m, src_row=src,
                          rec_list=lists, centroids=ct, centroids_rot=crot)
        return R.rslm_unpack_codes(plan, codes, m).cpu().numpy(), scales.cpu().numpy()

    c32 = cen.astype(np.float32)
    crot = R.rslm_fwht(plan, torch.from_numpy(c32).to(DEV)).cpu().numpy()
    hi = np.full(D, 0.05, np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
    a2 = torch.zeros((n, D), dtype=torch.uint8, device=DEV)
    a, sa = encode(t(x), t(c32), t(crot), t(np.arange(n)), t(assign.astype(np.int32)), t(-hi), t(hi), a2)
    src = np.full(n + 18, -1, dtype=np.int64)
    place = rng.permutation(n + 18)[:n]
    src[place] = np.arange(n)
    lists = np.zeros(n + 18, np.int32)
    lists[place] = assign
    b2 = off(np.zeros((n, D), np.uint8))
    b, sb = encode(off(x), off(c32), off(crot), t(src), t(lists), off(-hi), off(hi), b2, shift=1)
    assert np.array_equal(a, b[place]) and np.array_equal(sa, sb[place])
    assert np.array_equal(a2.cpu().numpy(), b2.cpu().numpy())
    unused = np.setdiff1d(np.arange(n + 18), place)
    assert not b[unused].any() and not sb[unused].any()


@pytest.mark.parametrize("D,bits", [(131, 4), (384, 4), (300, 3), (768, 2), (1100, 2), (513, 1)])
@pytest.mark.parametrize("shift", [1, 2, 3])
def test_codes_at_any_byte(R, D, bits, shift):
    plan = R.Plan(D, bits, passes=2)
    n = 45
    x = torch.from_numpy(synth.aniso(n, D, seed=D)).to(DEV)
    got = []
    for k in (0, shift):
        codes = torch.zeros(plan.code_bytes(n) + k, dtype=torch.uint8, device=DEV)[k:]
        scales = torch.zeros(n, dtype=torch.int32, device=DEV)
        R.rslm_encode(plan, x, codes, scales)
        got.append((codes, scales, R.rslm_decode(plan, codes, scales, n)))
    assert all(torch.equal(a, b) for a, b in zip(*got))
