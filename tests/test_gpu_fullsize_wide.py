"""Parity at a wide dimension, through the entry points the benchmark uses:
200,000 x 1,536 unit-norm anisotropic rows (the paper's 1,536-dimensional
text-embedding width), 256 lists, 4-bit RSLM with global scaling and two
rotation passes, SQ8 rescoring codes; a batch of 64 queries, nprobe = 16,
top-100 from the scan, top-10 after rescoring.

At this width the encoder spreads a vector's 12 blocks over four rows of lanes and
the scan scores each item in two passes of 24 chunks, keeping the partial
residual dot in the score slot between them.  The oracle checks what it can
compute one by one: the rotated queries and probe lists, assignment, codes
and scale codes of sampled vectors, and for two queries the returned top-k
against the oracle's scores of every member of all probed lists, and the
rescored shortlist.  Oracle inputs are the seeded rows (generated on the
host) and seeded centres; nothing the oracle consumes comes from the
library.
"""

import numpy as np
import pytest

import oracle
import synth
from tests import fullsize_common as F
from tests import helpers as H

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

WN, WD, WNLIST, WQ, WNPROBE, WK, WK_OUT = 200_000, 1536, 256, 64, 16, 100, 10


@pytest.fixture(scope="module")
def wide():
    import paper_2608_30384_amd as R
    from paper_2608_30384_amd import ivf

    dev = torch.device("cuda", 0)
    xh = synth.aniso(WN, WD, seed=41, normalize=True)
    x = torch.from_numpy(xh).to(dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(9)
    cen = x[torch.randperm(WN, generator=gen, device=dev)[:WNLIST]].clone()
    plan = R.Plan(WD, 4, passes=2, scale_mode="global")
    resid = torch.empty_like(x)
    index, _, assign = ivf.build_index(plan, x, cen, resid_rot=resid)
    codes2, lo, hi = ivf.build_sq8(resid)
    del resid
    q = synth.queries_like("aniso", WQ, WD, data_seed=41, query_seed=42)
    q = (q / np.linalg.norm(q, axis=1, keepdims=True)).astype(np.float32)
    qt = torch.from_numpy(q).to(dev)
    qrot = R.rslm_fwht(plan, qt)
    pid, pdot = R.ivf_assign_probe(qt, cen, WNPROBE, R.IVF_PROBE_IP)
    s1, i1 = R.rslm_scan_topk(plan, index, qrot, pid, pdot, WK)
    s2, i2 = R.rslm_rescore(codes2, lo, hi, qrot, s1, i1, WK_OUT)
    torch.cuda.synchronize()
    out = dict(R=R, plan=plan, xh=xh, cen=cen.cpu().numpy().astype(np.float64), q=q, cen_t=cen,
               crot=R.rslm_fwht(plan, cen), codes2=codes2, lo=lo.cpu().numpy(), hi=hi.cpu().numpy(),
               index=index, assign=assign.cpu().numpy(), pos=F.record_positions(torch, index, WN),
               qrot=qrot.cpu().numpy(), pid=pid.cpu().numpy(), pdot=pdot.cpu().numpy(),
               s1=s1.cpu().numpy(), i1=i1.cpu().numpy(), s2=s2.cpu().numpy(),
               i2=i2.cpu().numpy(), Rm=H.rot(WD, 2), C=synth.codebook(4))
    yield out
    del out
    torch.cuda.empty_cache()


def test_wide_rotation_and_probe(wide):
    f = wide
    qr = f["q"].astype(np.float64) @ f["Rm"].T
    assert np.all(np.abs(f["qrot"] - qr) <= 2e-6 * np.linalg.norm(f["q"], axis=1, keepdims=True))
    rid, _, dots = oracle.probe_ip(f["q"], f["cen"], WNPROBE)
    cmax = np.abs(f["cen"]).max()
    for i in range(WQ):
        tol = 1e-5 * np.linalg.norm(f["q"][i]) * cmax * np.sqrt(WD)
        assert np.all(np.abs(f["pdot"][i] - dots[i, f["pid"][i]]) <= tol)
        if set(f["pid"][i]) != set(rid[i]):
            srt = np.sort(dots[i])[::-1]
            assert srt[WNPROBE - 1] - srt[WNPROBE] <= 2 * tol


def test_wide_assign_and_encode_sampled(wide):
    f = wide
    ids = synth.random_rows(WN, 1500, seed=14)
    xs = f["xh"][ids].astype(np.float64)
    a, keep = F.check_assign(f["assign"][ids], xs, f["cen"])
    enc = oracle.encode(xs[keep], f["Rm"], f["C"], 4, centroids=f["cen"][a[keep]],
                        scale_mode="global")
    codes, sc = F.gpu_records(torch, f["R"], f["plan"], f["index"], f["pos"], ids[keep], 4, WD)
    ok = F.check_codes(codes, sc, enc, f["C"])
    assert ok.mean() > 0.98


@pytest.mark.parametrize("i", [5, 50])
def test_wide_scan_topk_sampled(wide, i):
    """Pairing and completeness over every member of all 16 probed lists."""
    f = wide
    gi, gs = f["i1"][i], f["s1"][i]
    F.check_topk_order(gs, gi, WK)
    qn = np.linalg.norm(f["q"][i])
    members, lst = F.members_of(torch, f["index"], f["pid"][i])
    xs = f["xh"][members].astype(np.float64)
    best = lst == f["pid"][i][0]
    a, _ = oracle.assign_l2_expanded(xs[best], f["cen"])
    assert (a == f["pid"][i][0]).mean() >= 0.99
    sm, xnm, near, _ = F.oracle_member_scores(xs, lst, f["cen"], f["q"][i], f["Rm"], f["C"], 4)
    F.check_probed(gs, gi, members, sm, H.score_tol(sm, qn, xnm), near)


@pytest.mark.parametrize("i", [5])
def test_wide_rescore_sampled(wide, i):
    """SQ8 records against the oracle's second residual; the rescoring
    against the decode of the stored records."""
    f = wide
    ri, rs = f["i2"][i], f["s2"][i]
    cand, s1 = f["i1"][i], f["s1"][i].astype(np.float64)
    assert set(ri.tolist()) <= set(cand.tolist())
    F.check_topk_order(rs, ri, WK_OUT)
    qr = f["q"][i].astype(np.float64) @ f["Rm"].T
    lo, hi = f["lo"].astype(np.float64), f["hi"].astype(np.float64)
    step = (hi - lo) / 255.0
    t = torch.from_numpy(cand.astype(np.int64)).to(f["codes2"].device)
    c2 = f["codes2"][t].cpu().numpy()
    xs = f["xh"][cand].astype(np.float64)
    a, _ = oracle.assign_l2_expanded(xs, f["cen"])
    enc1 = oracle.encode(xs, f["Rm"], f["C"], 4, centroids=f["cen"][a], scale_mode="global")
    err, r2, same, _ = F.r2_error(f["R"], torch, f["plan"], xs, a, f["cen_t"], f["crot"], f["Rm"],
                               enc1, f["C"], f["cen"])
    same &= f["assign"][cand] == a
    assert same.mean() >= 0.95
    bound = F.r2_bound(xs, f["cen"][a])
    assert np.all(err[same] <= bound[same]), (err / bound).max()
    dec = lo + c2 * step
    slack = 0.5 * step * (1 + 1e-4) + err[:, None]
    assert np.all(np.abs(dec - r2)[same] <= slack[same])
    s2 = s1 + dec @ qr
    ref_s, ref_i = oracle.topk(s2, cand, WK_OUT)
    tol = 1e-5 * (np.abs(s2).max() + np.linalg.norm(qr))
    H.check_topk(rs, ri, ref_s, ref_i, lambda v: np.full(np.shape(v), tol), s2, cand)
