"""Packed records from whole tiles: sizes around the record length where the
tile kernel starts, record lengths of every remainder mod 4, a ragged last
tile, and unaligned arrays, against the canonical codes and the scale words;
and the SQ8 ranges over row counts that split unevenly, against torch."""

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("D,bits,mode,lite", [
    (184, 4, "global", False), (188, 4, "local", False), (189, 4, "global", False), (300, 4, "local", False),
    (2049, 4, "local", False), (256, 4, "global", True), (230, 3, "global", False), (161, 3, "local", False),
    (240, 2, "global", False), (333, 2, "local", False), (481, 1, "global", False), (1601, 1, "local", False)])
@pytest.mark.parametrize("n,shift", [(1, 0), (16, 0), (333, 0), (50, 1)])
def test_pack_records(D, bits, mode, lite, n, shift):
    import paper_2608_30384_amd as R
    plan = R.Plan(D, bits, passes=1, scale_mode=mode, lite=lite)
    g = torch.Generator(device=DEV).manual_seed(D + n)
    raw = torch.randint(0, 256, (plan.code_bytes(n) + shift,), generator=g, device=DEV, dtype=torch.uint8)
    scales = torch.randint(0, 1 << 31, (n,), generator=g, device=DEV, dtype=torch.int64).to(torch.int32)
    tiles = raw[shift:]
    got = R.rslm_pack_records(plan, tiles, scales, n)
    canon = R.rslm_unpack_codes(plan, tiles, n)
    assert torch.equal(got[:, :plan.canon_bytes], canon)
    if not lite:
        suffix = scales.view(torch.uint8).view(n, 4)[:, :4 if mode == "global" else 2]
        assert torch.equal(got[:, plan.canon_bytes:], suffix)


@pytest.mark.parametrize("n,dim", [(1, 3), (63, 70), (129, 257), (70001, 5), (5000, 1100)])
def test_sq8_ranges(n, dim):
    import paper_2608_30384_amd as R
    v = torch.randn(n, dim, device=DEV)
    lo, hi = R.rslm_sq8_fit(v)
    assert torch.equal(lo, v.amin(0)) and torch.equal(hi, v.amax(0))
    w = torch.randn(17, dim, device=DEV) * 2
    R.rslm_sq8_fit(w, lo, hi, accumulate=True)
    both = torch.cat([v, w])
    assert torch.equal(lo, both.amin(0)) and torch.equal(hi, both.amax(0))
