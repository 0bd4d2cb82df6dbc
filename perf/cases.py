"""Representative workloads of the RSLM path, for timing and comparison.

The work a user has this framework do on one GPU, through its Python entry
points: answering batches of queries over an IVF index (rotate, probe, scan,
rescore), encoding vectors for an index, compressing and decompressing
stand-alone records, scoring one query against many records, and training the
partition.  Sizes are those of the benchmark's configurations and of the
paper's codec microbenchmarks; drawn cases spread over the same ranges, odd
dimensions and counts, every bit width, both scale modes and the Lite codec
among them.

Inputs are synthetic and made on the GPU from the seed: vectors are a mixture
around partition centres with a power-law variance spectrum and a shared
offset, partition sizes are log-normal, queries probe popular partitions more
often.  An index's codes are drawn directly with the distribution that the
rotation gives them (independent, the Lloyd-Max cells of a Gaussian), so that
an index of millions of records is ready in a fraction of a second and does
not depend on the encoder.
"""

import math

import numpy as np
import torch

import paper_2608_30384_amd as R
import synth
from paper_2608_30384_amd import ivf

RESID = 0.7  # norm of a vector's residual to its centre (the centres: about 0.9)


def listed():
    return [
        # The smallest call: one query over a 10,000-vector collection, where
        # launches and the latency of each stage count.
        dict(name="search_tiny128", kind="search", n=10_000, dim=128, bits=2, passes=1,
             scale="global", lite=False, nlist=16, nprobe=4, batch=1, k=10, rescore="none", k_out=0),
        # An ordinary low-dimensional collection served in batches.
        dict(name="search_mid96", kind="search", n=1_000_000, dim=96, bits=4, passes=2,
             scale="global", lite=False, nlist=1024, nprobe=32, batch=256, k=100, rescore="sq8",
             k_out=10),
        # Text embeddings: the benchmark's configuration.
        dict(name="search_text768", kind="search", n=10_000_000, dim=768, bits=4, passes=2,
             scale="global", lite=False, nlist=4096, nprobe=64, batch=256, k=100, rescore="sq8",
             k_out=10),
        # Lowest-memory codes at the bit-width sweep's dimension: 1 bit, no
        # rescoring records.
        dict(name="search_sweep1024_b1", kind="search", n=10_000_000, dim=1024, bits=1, passes=2,
             scale="global", lite=False, nlist=4096, nprobe=64, batch=256, k=10, rescore="none",
             k_out=0),
        # Large batches over large lists with 2-bit RSLM rescoring records (the
        # capacity configuration's list and batch sizes on a part of its lists).
        dict(name="search_capacity768", kind="search", n=20_000_000, dim=768, bits=4, passes=2,
             scale="global", lite=False, nlist=4096, nprobe=128, batch=1024, k=100,
             rescore="rslm2", k_out=10),
        # Adding vectors to an index: scan records and SQ8 rescoring codes.
        dict(name="encode_text768_sq8", kind="encode", n=65_536, dim=768, bits=4, passes=2,
             scale="global", lite=False, nlist=4096, second="sq8"),
        # Building the capacity index block by block: both stages' records.
        dict(name="encode_capacity768_2st", kind="encode", n=524_288, dim=768, bits=4, passes=2,
             scale="global", lite=False, nlist=16_384, second="rslm2"),
        # Low-bit codes (2-D codebook) at the bit-width sweep's dimension.
        dict(name="encode_sweep1024_b2", kind="encode", n=65_536, dim=1024, bits=2, passes=2,
             scale="global", lite=False, nlist=4096, second="none"),
        # The paper's compression microbenchmark: D = 2,049, stand-alone records.
        dict(name="compress2049", kind="compress", n=65_536, dim=2049, bits=4, passes=-1,
             scale="local", lite=False),
        # Reading vectors back out of an index.
        dict(name="decompress768", kind="decompress", n=65_536, dim=768, bits=4, passes=2,
             scale="global", lite=False, nlist=4096),
        # The paper's OneToMany microbenchmark: one query, 16.8 M records.
        dict(name="onetomany256", kind="score", pool=16_777_216, n=16_777_216, gathered=False,
             dim=256, bits=4, passes=-1, scale="local", lite=False, batch=1),
        # One Lloyd iteration of the text-embedding partition's training.
        dict(name="kmeans_text768", kind="kmeans", n=1_048_576, dim=768, nlist=4096),
    ]


# ------------------------------------------------------------------ drawn cases
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dim(rng):
    if rng.random() < 0.65:
        return rng.choice([64, 96, 100, 128, 200, 256, 300, 384, 512, 768, 960, 1024, 1536])
    return rng.randint(48, 1600)


def _codec(rng, dim):
    bits = rng.choice([1, 2, 3, 4, 4])
    return dict(dim=dim, bits=bits, passes=-1, scale=rng.choice(["local", "global", "global"]),
                lite=bits == 4 and dim >= 64 and rng.random() < 0.2)


def draw(rng):
    kind = rng.choice(["search"] * 5 + ["encode"] * 3 + ["compress", "decompress", "score", "kmeans"])
    dim = _dim(rng)
    if kind == "search":
        n = _log(rng, 10_000, 4_000_000)
        nlist = max(8, min(8192, _log(rng, 1, 4) * int(math.sqrt(n) / 2)))
        nprobe = max(1, min(128, nlist // 4, _log(rng, 4, 128)))
        k = rng.choice([1, 10, 50, 100, 200])
        c = _codec(rng, dim)
        rescore = rng.choice(["none", "sq8", "sq8", "none" if c["lite"] else "rslm2"])
        return dict(kind=kind, n=n, **c, nlist=nlist, nprobe=nprobe, batch=_log(rng, 1, 600), k=k,
                    rescore=rescore, k_out=0 if rescore == "none" else max(1, k // 10))
    if kind == "encode":
        c = _codec(rng, dim)
        second = rng.choice(["none", "sq8", "fit", "none" if c["lite"] else "rslm2"])
        return dict(kind=kind, n=_log(rng, 500, 200_000_000 // dim), **c, nlist=_log(rng, 16, 8192),
                    second=second)
    if kind == "compress":
        return dict(kind=kind, n=_log(rng, 500, 130_000_000 // dim), **_codec(rng, dim))
    if kind == "decompress":
        return dict(kind=kind, n=_log(rng, 500, 100_000_000 // dim), **_codec(rng, dim),
                    nlist=rng.choice([0, _log(rng, 16, 8192)]))
    if kind == "score":
        pool = _log(rng, 10_000, 2_000_000_000 // dim)
        gathered = rng.random() < 0.5
        batch = rng.choice([1, 1, 1, rng.randint(2, 12)])
        return dict(kind=kind, pool=pool, n=pool if not gathered else max(1, pool // rng.choice([1, 2, 8])),
                    gathered=gathered, **_codec(rng, dim), batch=batch)
    nlist = _log(rng, 16, 8192)
    most = min(4_000_000, 5_000_000_000_000 // (2 * dim * nlist))
    return dict(kind=kind, n=max(4 * nlist, _log(rng, 4_000, most)), dim=dim, nlist=nlist)


# ------------------------------------------------------------------ inputs
DEV = "cuda"


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, device=DEV)


def _spectrum(dim):
    var = 1.0 / np.arange(1, dim + 1)
    return torch.tensor(np.sqrt(var / var.sum()), dtype=torch.float32, device=DEV)


def _centres(gen, nlist, dim):
    mu = _randn(gen, dim)
    mu = 0.5 * mu / mu.norm()
    return (mu + math.sqrt(1 - RESID ** 2) * _spectrum(dim) * _randn(gen, nlist, dim)).contiguous()


def _around(gen, centres, assign):
    out = _randn(gen, assign.numel(), centres.shape[1])
    return out.mul_(RESID * _spectrum(centres.shape[1])).add_(centres[assign])


def _list_sizes(seed, n, nlist):
    """Log-normal partition sizes (sigma 0.5) that add up to n: the same sizes for
    every seed, dealt to other partitions."""
    z = np.random.default_rng([nlist, 1]).standard_normal(nlist)
    w = np.exp(0.5 * z)
    sizes = np.floor(w / w.sum() * n).astype(np.int64)
    sizes[:n - int(sizes.sum())] += 1
    return np.random.default_rng([int(seed), 2]).permutation(sizes)


def _members(gen, sizes):
    """The partition of each vector, in random order."""
    lists = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), torch.tensor(sizes, device=DEV))
    return lists[torch.randperm(lists.numel(), generator=gen, device=DEV)]


def _plan(c):
    return R.Plan(c["dim"], c["bits"], passes=c["passes"], scale_mode=c["scale"], lite=c["lite"])


def _lead(c):
    return 0 if not c["lite"] else 32 if c["scale"] == "global" else 16


def _gauss_cells(bits):
    """Probability of each 1-D Lloyd-Max cell under a standard normal."""
    cb = synth.codebook(bits)[:, 0].astype(np.float64)
    cdf = [0.0] + [0.5 * (1 + math.erf(t / math.sqrt(2))) for t in (cb[1:] + cb[:-1]) / 2] + [1.0]
    return np.diff(cdf)


def _quantile_table(prob):
    """65,536 equally likely entries with the given distribution."""
    edges = np.round(np.cumsum(prob) * 65536).astype(np.int64)
    return torch.tensor(np.searchsorted(edges, np.arange(65536), side="right").clip(max=len(prob) - 1),
                        dtype=torch.uint8, device=DEV)


def _draw_table(gen, table, n, width):
    out = torch.empty((n, width), dtype=torch.uint8, device=DEV)
    step = max(1, (1 << 26) // width)
    for lo in range(0, n, step):
        m = min(n, lo + step) - lo
        out[lo:lo + m] = table[torch.randint(0, 65536, (m, width), generator=gen, device=DEV,
                                             dtype=torch.int32)]
    return out


def _random_bytes(gen, n, width):
    return torch.randint(0, 256, (n, width), generator=gen, device=DEV, dtype=torch.uint8)


def _float_code(v, mbits, bias):
    """The 16-bit unsigned float code (mbits of mantissa) nearest below v."""
    b = v.float().contiguous().view(torch.int32) >> (23 - mbits)
    return b - ((127 - bias) << mbits)


def _float_value(u, mbits, bias):
    u = u.to(torch.int64)
    v = torch.ldexp(1.0 + (u & ((1 << mbits) - 1)).double() / (1 << mbits),
                    (u >> mbits) - bias)
    return torch.where(u == 0, torch.zeros_like(v), v)


def _scales(gen, c, n, norm):
    """Scale words (UE7M9 | UE4M12 << 16) of n records of residual norm about `norm`."""
    s = norm / math.sqrt(c["dim"]) * torch.exp(0.2 * _randn(gen, n))
    g = torch.full((n,), 1.0, device=DEV)
    if c["scale"] == "global":
        g = torch.exp(0.01 * _randn(gen, n))
    return (_float_code(s, 9, 63) | (_float_code(g, 12, 7) << 16)).contiguous()


def _canonical(gen, c, n, scales):
    """n random records in the canonical bit order, n x canonical bytes."""
    dim, bits = c["dim"], c["bits"]
    if bits == 3:
        width = -(-dim // 8) * 8
        sym = _draw_table(gen, _quantile_table(_gauss_cells(3)), n, width)
        sym[:, dim:] = 0
        out = torch.empty((n, width // 8 * 3), dtype=torch.uint8, device=DEV)
        step = max(1, (1 << 26) // width)
        shift = 3 * torch.arange(8, device=DEV, dtype=torch.int32)
        for lo in range(0, n, step):
            w = (sym[lo:lo + step].view(-1, width // 8, 8).to(torch.int32) << shift).sum(-1, dtype=torch.int32)
            out[lo:lo + step] = torch.stack([w & 255, (w >> 8) & 255, w >> 16], -1).view(
                -1, width // 8 * 3).to(torch.uint8)
        return out[:, :-(-3 * dim // 8)].contiguous()
    n_sym = dim if bits == 4 else -(-dim // (4 if bits == 1 else 2))
    width = (n_sym + 1) // 2
    if bits == 4:
        p = _gauss_cells(4)
        out = _draw_table(gen, _quantile_table(np.outer(p, p).reshape(-1)), n, width)
    else:
        out = _random_bytes(gen, n, width)
    if n_sym % 2:
        out[:, -1] &= 15
    lead = _lead(c)
    if lead:  # 3-bit leading codes, bit j of the scale word in coordinate j's top bit
        j = torch.arange(0, lead, 2, device=DEV, dtype=torch.int32)
        sc = scales[:, None]
        top = (((sc >> j) & 1) << 3) | (((sc >> (j + 1)) & 1) << 7)
        out[:, :lead // 2] = (out[:, :lead // 2] & 0x77) | top.to(torch.uint8)
    return out


def _index_data(c, seed, gen):
    sizes = _list_sizes(seed, c["n"], c["nlist"])
    padded = (sizes + 15) // 16 * 16
    offsets = np.cumsum(padded) - padded
    total = int(padded.sum())
    centres = _centres(gen, c["nlist"], c["dim"])
    sizes_t = torch.tensor(sizes, device=DEV)
    pick = torch.multinomial(sizes_t.double(), c["batch"], replacement=True, generator=gen)
    queries = _around(gen, centres, pick)
    offsets_t = torch.tensor(offsets, device=DEV)
    live = torch.arange(total, device=DEV)
    owner = torch.repeat_interleave(torch.arange(c["nlist"], device=DEV), torch.tensor(padded, device=DEV))
    live = live - offsets_t[owner] < sizes_t[owner]
    ids = torch.full((total,), -1, dtype=torch.int32, device=DEV)
    ids[live] = torch.randperm(c["n"], generator=gen, device=DEV).to(torch.int32)
    scales = _scales(gen, c, total, RESID)
    canon = _canonical(gen, c, total, scales)
    return centres, queries, offsets_t, sizes_t, ids, scales, canon, int(sizes.max())


def _rescore_data(c, gen):
    n, dim = c["n"], c["dim"]
    if c["rescore"] == "sq8":  # residual codes, bell-shaped over the fitted range
        hi = 0.35 * RESID / math.sqrt(dim) * torch.exp(0.1 * _randn(gen, dim))
        p = np.exp(-0.5 * ((np.arange(256) - 127.5) / 28) ** 2)
        return dict(lo=-hi, hi=hi, codes2=_draw_table(gen, _quantile_table(p / p.sum()), n, dim))
    if c["rescore"] == "rslm2":
        c2 = dict(dim=dim, bits=2, scale="global", lite=False)
        return dict(scales2=_scales(gen, c2, n, 0.1 * RESID), codes2=_canonical(gen, c2, n, None))
    return {}


def _encode_data(c, seed, gen):
    centres = _centres(gen, c["nlist"], c["dim"])
    assign = _members(gen, _list_sizes(seed, c["n"], c["nlist"]))
    return centres, assign, _around(gen, centres, assign)


def _records_data(c, gen, n):
    scales = _scales(gen, c, n, 1.0)
    return scales, _canonical(gen, c, n, scales)


def prepare(case, seed):
    return dict(globals()["_prepare_" + case["kind"]](case, seed, _gen(seed)), case=case)


def _prepare_search(c, seed, gen):
    plan = _plan(c)
    centres, q, offsets, sizes, ids, scales, canon, most = _index_data(c, seed, gen)
    codes = R.rslm_pack_codes(plan, canon, ids.numel())
    index = R.Index(offsets, sizes.to(torch.int32), ids, codes, scales, max_list_size=most)
    s = dict(plan=plan, centres=centres, q=q, index=index, **_rescore_data(c, gen))
    if c["rescore"] == "rslm2":
        s["plan2"] = R.Plan(c["dim"], 2, passes=0, scale_mode="global")
    return s


def _prepare_encode(c, seed, gen):
    plan = _plan(c)
    centres, assign, x = _encode_data(c, seed, gen)
    _, _, src_row, rec_list, _, total = ivf.layout(assign, c["nlist"])
    s = dict(plan=plan, centres=centres, x=x, src_row=src_row, rec_list=rec_list, total=total,
             cen_rot=R.rslm_fwht(plan, centres),
             codes=torch.zeros(plan.code_bytes(total), dtype=torch.uint8, device=DEV),
             scales=torch.zeros(total, dtype=torch.int32, device=DEV))
    n, dim = x.shape
    if c["second"] == "sq8":
        hi = 0.6 * RESID / math.sqrt(dim) * torch.exp(0.1 * _randn(gen, dim))
        s.update(lo=-hi, hi=hi, codes2=torch.zeros((n, dim), dtype=torch.uint8, device=DEV))
    elif c["second"] == "rslm2":
        plan2 = R.Plan(dim, 2, passes=0, scale_mode="global")
        s.update(plan2=plan2, scales2=torch.zeros(n, dtype=torch.int32, device=DEV),
                 codes2=torch.zeros((n, plan2.canon_bytes), dtype=torch.uint8, device=DEV))
    elif c["second"] == "fit":
        s.update(resid=torch.zeros_like(x))
    return s


def _compress_input(c, gen):
    return _randn(gen, c["n"], c["dim"]).mul_(_spectrum(c["dim"])).add_(0.3 / math.sqrt(c["dim"]))


def _prepare_compress(c, seed, gen):
    plan = _plan(c)
    return dict(plan=plan, x=_compress_input(c, gen),
                codes=torch.zeros(plan.code_bytes(c["n"]), dtype=torch.uint8, device=DEV),
                scales=torch.zeros(c["n"], dtype=torch.int32, device=DEV))


def _decompress_data(c, seed, gen):
    scales, canon = _records_data(c, gen, c["n"])
    centres = rec_list = None
    if c["nlist"]:
        centres = _centres(gen, c["nlist"], c["dim"])
        rec_list = _members(gen, _list_sizes(seed, c["n"], c["nlist"])).to(torch.int32)
    return scales, canon, centres, rec_list


def _prepare_decompress(c, seed, gen):
    plan = _plan(c)
    scales, canon, centres, rec_list = _decompress_data(c, seed, gen)
    return dict(plan=plan, scales=scales, codes=R.rslm_pack_codes(plan, canon, c["n"]),
                centres=centres, rec_list=rec_list)


def _score_data(c, gen):
    scales, canon = _records_data(c, gen, c["pool"])
    q = _randn(gen, c["batch"], c["dim"]).mul_(_spectrum(c["dim"]))
    ids = torch.randint(0, c["pool"], (c["n"],), generator=gen, device=DEV) if c["gathered"] else None
    return scales, canon, q, ids


def _prepare_score(c, seed, gen):
    plan = _plan(c)
    scales, canon, q, ids = _score_data(c, gen)
    if c["lite"]:
        records = canon
    else:
        tail = scales.view(torch.uint8).view(-1, 4)[:, :4 if c["scale"] == "global" else 2]
        records = torch.cat([canon, tail], 1)
    return dict(plan=plan, records=records.contiguous(), q=q, ids=ids)


def _prepare_kmeans(c, seed, gen):
    x, centres = _kmeans_data(c, seed, gen)
    return dict(x=x, centres=centres)


def _kmeans_data(c, seed, gen):
    true = _centres(gen, c["nlist"], c["dim"])
    x = _around(gen, true, _members(gen, _list_sizes(seed, c["n"], c["nlist"])))
    first = torch.randperm(c["n"], generator=gen, device=DEV)[:c["nlist"]]
    return x, x[first].contiguous()


# ------------------------------------------------------------------ one pass
def run(state):
    return globals()["_run_" + state["case"]["kind"]](state, state["case"])


def _run_search(s, c):
    q_rot = R.rslm_fwht(s["plan"], s["q"])
    probe_ids, probe_dots = R.ivf_assign_probe(s["q"], s["centres"], c["nprobe"], R.IVF_PROBE_IP)
    scores, ids = R.rslm_scan_topk(s["plan"], s["index"], q_rot, probe_ids, probe_dots, c["k"])
    out = dict(scores=scores, ids=ids)
    if c["rescore"] == "sq8":
        out["scores2"], out["ids2"] = R.rslm_rescore(s["codes2"], s["lo"], s["hi"], q_rot, scores, ids,
                                                     c["k_out"])
    elif c["rescore"] == "rslm2":
        out["scores2"], out["ids2"] = R.rslm_rescore_rslm(s["plan2"], s["codes2"], s["scales2"], q_rot,
                                                          scores, ids, c["k_out"])
    return out


def _run_encode(s, c):
    kw = dict(n_records=s["total"], src_row=s["src_row"], rec_list=s["rec_list"],
              centroids=s["centres"], centroids_rot=s["cen_rot"])
    out = dict(codes=s["codes"], scales=s["scales"])
    if c["second"] == "sq8":
        R.rslm_encode_sq8(s["plan"], s["x"], s["codes"], s["scales"], s["lo"], s["hi"], s["codes2"], **kw)
        out["codes2"] = s["codes2"]
    elif c["second"] == "rslm2":
        R.rslm_encode_two_stage(s["plan"], s["plan2"], s["x"], s["codes"], s["scales"], s["codes2"],
                                s["scales2"], **kw)
        out.update(codes2=s["codes2"], scales2=s["scales2"])
    elif c["second"] == "fit":
        R.rslm_encode(s["plan"], s["x"], s["codes"], s["scales"], resid_rot=s["resid"], **kw)
        codes2, lo, hi = ivf.build_sq8(s["resid"])
        out.update(lo=lo, hi=hi, codes2=codes2)
    else:
        R.rslm_encode(s["plan"], s["x"], s["codes"], s["scales"], **kw)
    return out


def _run_compress(s, c):
    R.rslm_encode(s["plan"], s["x"], s["codes"], s["scales"])
    return R.rslm_pack_records(s["plan"], s["codes"], s["scales"], c["n"])


def _run_decompress(s, c):
    return R.rslm_decode(s["plan"], s["codes"], s["scales"], c["n"], rec_list=s["rec_list"],
                         centroids=s["centres"])


def _run_score(s, c):
    q_rot = R.rslm_fwht(s["plan"], s["q"])
    return R.rslm_score(s["plan"], s["records"], q_rot, ids=s["ids"])


def _run_kmeans(s, c):
    assign, dist = R.ivf_assign_probe(s["x"], s["centres"], 1, R.IVF_ASSIGN_L2)
    centres = R.ivf_kmeans_update(s["x"], assign, s["centres"].clone())
    return dict(assign=assign, dist=dist, centres=centres)


# ------------------------------------------------------------------ what a pass cannot do without
def _canon_bytes(dim, bits):
    n_sub = -(-dim // {1: 4, 2: 2, 3: 1, 4: 1}[bits])
    return -(-n_sub * (3 if bits == 3 else 4) // 8)


def _record(c):
    return _canon_bytes(c["dim"], c["bits"]) + (0 if c["lite"] else 4 if c["scale"] == "global" else 2)


def work(case):
    c = case
    kind, dim = c["kind"], c["dim"]
    if kind == "search":
        q, pairs = c["batch"], c["batch"] * c["nprobe"] * (c["n"] / c["nlist"])
        # the share of the lists that a batch touches, were its probes independent
        share = 1 - (1 - c["nprobe"] / c["nlist"]) ** q
        b = share * c["n"] * (_record(c) + 4) + 4 * c["nlist"] * dim + 4 * q * dim + 8 * q * c["k"]
        if c["rescore"] != "none":
            b += q * c["k"] * (dim if c["rescore"] == "sq8" else _canon_bytes(dim, 2) + 4)
        return dict(bytes=b, flops=2 * dim * (pairs + q * c["nlist"]))
    if kind == "encode":
        b = 4 * dim + _record(c) + 16
        b += {"none": 0, "sq8": dim, "rslm2": _canon_bytes(dim, 2) + 4, "fit": 5 * dim}[c["second"]]
        return dict(bytes=c["n"] * b, flops=c["n"] * dim * 40)
    if kind == "compress":
        return dict(bytes=c["n"] * (4 * dim + _record(c)), flops=c["n"] * dim * 30)
    if kind == "decompress":
        return dict(bytes=c["n"] * (4 * dim + _record(c) + 4), flops=c["n"] * dim * 20)
    if kind == "score":
        return dict(bytes=c["n"] * (_record(c) + 4 * c["batch"] + (8 if c["gathered"] else 0)),
                    flops=2 * c["n"] * dim * c["batch"])
    return dict(bytes=2 * 4 * dim * (c["n"] + c["nlist"]), flops=2 * c["n"] * dim * c["nlist"])


def tolerance(case):
    return TOLERANCE[case["kind"]]


# About four times what float32 sums in another order show against 64 bits.
# Whole values: codes differ where a coordinate or a scale is at a rounding
# midpoint (a scale code has 10 or 13 significant bits, so about one in a
# thousand is within a float32 rounding of one), ids where two scores or
# distances are equal to float32 precision; a vector that moves to a centre at
# the same distance moves both centres' means.
TOLERANCE = {
    "search": {"rel": 3e-6, "max": 1e-5, "differ": 0.01},
    "encode": {"rel": 1e-4, "max": 2e-3, "differ": 2e-3},
    "compress": {"rel": 0.0, "differ": 5e-4},
    "decompress": {"rel": 6e-7, "max": 4e-6},
    "score": {"rel": 1e-6, "max": 8e-6},
    "kmeans": {"rel": 1.2e-3, "max": 0.4, "differ": 5e-5},
}


# ------------------------------------------------------------------ the same in 64 bits
def _passes(c):
    return c["passes"] if c["passes"] >= 0 else 1 if c["bits"] == 4 and c["dim"] <= 256 else 2


def _rotate64(v, passes, inverse=False):
    """Rows of v times the rotation (or its transpose), by explicit Hadamard products."""
    y = v.double().clone()
    dim = y.shape[1]
    if passes == 0:
        return y
    size = 128 if dim >= 128 else 1 << (dim.bit_length() - 1)
    h = torch.ones((1, 1), dtype=torch.float64, device=y.device)
    while h.shape[0] < size:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)], 0)
    h = h / math.sqrt(size)
    blocks = [b * size for b in range(dim // size)] + ([dim - size] if dim % size else [])
    sign = torch.tensor(synth.sign_table().astype(np.float64), device=y.device)
    at = torch.arange(dim, device=y.device)
    perm = synth.permutation_table()
    if size < 128:
        bits = size.bit_length() - 1
        perm = np.array([int(format(k, "0%db" % bits)[::-1], 2) if bits else 0 for k in range(size)])
    m = dim // size
    source = np.arange(dim)
    for b in range(m):
        source[np.arange(size) * m + b] = b * size + np.asarray(perm)
    source = torch.tensor(source, device=y.device)

    def block_pass(y, order):
        for o in order:
            y[:, o:o + size] = y[:, o:o + size] @ h
        return y

    if not inverse:
        y = block_pass(y * sign[at % 256], blocks)
        if passes == 2:
            y = block_pass(y[:, source] * sign[(at + 127) % 256], blocks)
        return y
    if passes == 2:
        y = block_pass(y, blocks[::-1]) * sign[(at + 127) % 256]
        back = torch.empty_like(y)
        back[:, source] = y
        y = back
    return block_pass(y, blocks[::-1]) * sign[at % 256]


def _symbols(c, canon):
    if c["bits"] == 3:
        n, width = canon.shape
        pad = torch.zeros((n, -width % 3), dtype=torch.uint8, device=canon.device)
        w = torch.cat([canon, pad], 1).view(n, -1, 3).to(torch.int32)
        w = w[..., 0] | (w[..., 1] << 8) | (w[..., 2] << 16)
        shift = 3 * torch.arange(8, device=canon.device, dtype=torch.int32)
        return ((w[..., None] >> shift) & 7).view(n, -1)
    return torch.stack([canon & 15, canon >> 4], -1).view(canon.shape[0], -1).to(torch.int32)


def _decoded64(c, canon):
    """The centroid values of canonical records, n x dim."""
    sym = _symbols(c, canon)
    cb = torch.tensor(synth.codebook(c["bits"]).astype(np.float64), device=canon.device)
    n_sub = -(-c["dim"] // cb.shape[1])
    lead = _lead(c)
    if lead:
        cb3 = torch.tensor(synth.codebook(3)[:, 0].astype(np.float64), device=canon.device)
        head = cb3[(sym[:, :lead] & 7).long()]
        return torch.cat([head, cb[sym[:, lead:n_sub].long(), 0]], 1)
    return cb[sym[:, :n_sub].long()].reshape(canon.shape[0], -1)[:, :c["dim"]]


def _rows64(c):
    """Rows worked on at once: float64 temporaries of 256 MB."""
    return max(1, (1 << 25) // c["dim"])


def _dots64(q, v):
    return torch.stack([(v * one).sum(1) for one in q]) if len(q) < 4 else q @ v.contiguous().T


def _scale64(c, scales):
    s = _float_value(scales & 0xffff, 9, 63)
    g = _float_value((scales >> 16) & 0xffff, 12, 7) if c["scale"] == "global" else torch.ones_like(s)
    return s, g


def _best(scores, ids, k):
    top, at = scores.topk(min(k, scores.shape[1]), dim=1)
    got = torch.gather(ids, 1, at)
    got = torch.where(top == -math.inf, torch.full_like(got, -1), got)
    if top.shape[1] < k:
        fill = (top.shape[0], k - top.shape[1])
        top = torch.cat([top, top.new_full(fill, -math.inf)], 1)
        got = torch.cat([got, got.new_full(fill, -1)], 1)
    return top, got


def exact(case, seed):
    fn = globals().get("_exact_" + case["kind"])
    return None if fn is None else fn(case, seed, _gen(seed))


def _exact_search(c, seed, gen):
    centres, q, offsets, sizes, ids, scales, canon, most = _index_data(c, seed, gen)
    q_rot = _rotate64(q, _passes(c))
    dots, probes = (q.double() @ centres.double().T).topk(c["nprobe"], dim=1)
    sc, gl = _scale64(c, scales)
    all_scores = torch.full((c["batch"], c["nprobe"], most), -math.inf, dtype=torch.float64, device=DEV)
    wanted = {}
    for i, row in enumerate(probes.tolist()):
        for j, p in enumerate(row):
            wanted.setdefault(p, []).append((i, j))
    offs, szs, step = offsets.tolist(), sizes.tolist(), _rows64(c)
    for p, pairs in wanted.items():
        lo, m = offs[p], szs[p]
        qi, pj = (torch.tensor(v, device=DEV) for v in zip(*pairs))
        for a in range(0, m, step):
            r = slice(lo + a, lo + min(m, a + step))
            part = _dots64(q_rot[qi], _decoded64(c, canon[r]))
            all_scores[qi, pj, a:a + part.shape[1]] = gl[r] * (dots[qi, pj][:, None] + sc[r] * part)
    del canon
    flat = all_scores.view(c["batch"], -1)
    top, at = flat.topk(min(c["k"], flat.shape[1]), dim=1)
    rec = offsets[torch.gather(probes, 1, at // most)] + at % most
    scores, got = _best(top, ids[rec.clamp(max=ids.numel() - 1)], c["k"])
    out = dict(scores=scores, ids=got)
    if c["rescore"] != "none":
        d = _rescore_data(c, gen)
        rows = got.clamp(min=0).long()
        if c["rescore"] == "sq8":
            lo, step = d["lo"].double(), (d["hi"].double() - d["lo"].double()) / 255
            dot = torch.stack([(lo + step * d["codes2"][r].double()) @ v for r, v in zip(rows, q_rot)])
            s2 = scores + dot
        else:
            c2 = dict(c, bits=2, lite=False, scale="global")
            dot = torch.stack([_decoded64(c2, d["codes2"][r]) @ v for r, v in zip(rows, q_rot)])
            a, b = _scale64(c2, d["scales2"][rows])
            s2 = b * (scores + a * dot)
        s2 = torch.where(got < 0, torch.full_like(s2, -math.inf), s2)
        out["scores2"], out["ids2"] = _best(s2, got, c["k_out"])
    return out


def _exact_encode(c, seed, gen):
    """The ranges of the rotated second residual; codes have no 64-bit value."""
    if c["second"] != "fit":
        return None
    centres, assign, x = _encode_data(c, seed, gen)
    cb = torch.tensor(synth.codebook(c["bits"]).astype(np.float64), device=DEV)
    lead = _lead(c)
    resid = torch.empty(x.shape, dtype=torch.float64, device=DEV)
    t = np.linspace(0, 12, 200_001)
    cdf = np.array([math.erf(v / math.sqrt(2)) for v in t]) ** c["dim"]
    emax = float(np.sum((1 - cdf)[1:] + (1 - cdf)[:-1]) / 2 * (t[1] - t[0]))
    g = cb.shape[1]
    for lo in range(0, x.shape[0], 1 << 12):
        xs, cs = x[lo:lo + (1 << 12)].double(), centres[assign[lo:lo + (1 << 12)]].double()
        z = _rotate64(xs - cs, _passes(c))
        u = z * (emax / z.abs().amax(1, keepdim=True))
        pad = torch.zeros((len(u), -c["dim"] % g), dtype=torch.float64, device=DEV)
        sub = torch.cat([u, pad], 1).view(len(u), -1, g)
        near = (sub.reshape(-1, g) @ cb.T - (cb * cb).sum(1) / 2).argmax(1)
        hat = cb[near].view(len(u), -1)[:, :c["dim"]].clone()
        if lead:
            cb3 = torch.tensor(synth.codebook(3)[:, 0].astype(np.float64), device=DEV)
            hat[:, :lead] = cb3[(u[:, :lead, None] - cb3).abs().argmin(-1)]
        s = _round_code(z.norm(dim=1) / hat.norm(dim=1), 9)
        base = _rotate64(cs, _passes(c)) + s[:, None] * hat
        gl = torch.ones_like(s)
        if c["scale"] == "global":
            gl = _round_code(xs.norm(dim=1) / base.norm(dim=1), 12)
        resid[lo:lo + len(u)] = _rotate64(xs, _passes(c)) - gl[:, None] * base
    return dict(codes=None, scales=None, lo=resid.amin(0), hi=resid.amax(0), codes2=None)


def _round_code(v, mbits):
    m, e = torch.frexp(v)
    return torch.ldexp(torch.round(m * (1 << (mbits + 1))), e - (mbits + 1))


def _exact_decompress(c, seed, gen):
    scales, canon, centres, rec_list = _decompress_data(c, seed, gen)
    s, g = _scale64(c, scales)
    out = torch.empty((c["n"], c["dim"]), dtype=torch.float64, device=DEV)
    step = _rows64(c)
    for lo in range(0, c["n"], step):
        r = slice(lo, min(c["n"], lo + step))
        v = _rotate64(s[r, None] * _decoded64(c, canon[r]), _passes(c), inverse=True)
        if centres is not None:
            v += centres[rec_list[r].long()].double()
        out[r] = g[r, None] * v
    return out


def _exact_score(c, seed, gen):
    scales, canon, q, ids = _score_data(c, gen)
    q_rot = _rotate64(q, _passes(c))
    s, g = _scale64(c, scales)
    out = torch.empty((c["batch"], c["pool"]), dtype=torch.float64, device=DEV)
    step = _rows64(c)
    for lo in range(0, c["pool"], step):
        r = slice(lo, lo + step)
        out[:, r] = g[r] * s[r] * _dots64(q_rot, _decoded64(c, canon[r]))
    return out if ids is None else out[:, ids]


def _exact_kmeans(c, seed, gen):
    x, centres = _kmeans_data(c, seed, gen)
    c64 = centres.double()
    assign = torch.empty(c["n"], dtype=torch.int64, device=DEV)
    dist = torch.empty(c["n"], dtype=torch.float64, device=DEV)
    sums = torch.zeros_like(c64)
    for lo in range(0, c["n"], 1 << 13):
        xs = x[lo:lo + (1 << 13)].double()
        d = (xs * xs).sum(1)[:, None] - 2 * (xs @ c64.T) + (c64 * c64).sum(1)
        dist[lo:lo + len(xs)], assign[lo:lo + len(xs)] = d.min(1)
        sums.index_add_(0, assign[lo:lo + len(xs)], xs)
    count = torch.bincount(assign, minlength=c["nlist"])[:, None]
    return dict(assign=assign, dist=dist, centres=torch.where(count > 0, sums / count.clamp(min=1), c64))
