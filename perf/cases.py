"""The detector's work as a user's program asks for it, one call sequence a kind.

step    one live pass, its Eq. 4 scores and their AUROC (canary_sim, drift_score,
        auroc, auroc_values)
batch   several runs over one reference set in batched launches (canary_sim_batch,
        drift_score_batch, auroc_launch, auroc_values)
score   Eq. 4 alone on activations the peers returned (drift_score)
ablate  the metric ablations on arrays in hand (drift_score_f16ref, cosine_score,
        cosine_score_f16ref)
table1  one attack of the paper's main table: the exact-norm scale, the live pass
        and an independent benign recompute, every detector setting and its ranking
chain   a substudy configuration with the live error carried between stages
fused   the simulation study's live pass and Eq. 4 in one launch (sim_score)
rank    the AUROC of score tables in hand, in total and per canary
refs    the verifier's offline pass: references, their statistics and scales

S shards, C canaries, T tokens, H hidden; arrays as in include/cdt.h.
"""
import math

import numpy as np
import torch

from paper_2607_19490_amd import cdt

DEV = "cuda"
TAMPERS = {"add": cdt.T_ADD, "flip": cdt.T_FLIP, "scale": cdt.T_SCALE,
           "mixed": cdt.T_ADD | cdt.T_FLIP | cdt.T_SCALE}
RANK_ALL = cdt.AUROC_CONTROL | cdt.AUROC_POOLED | cdt.AUROC_RANDOM


def listed():
    def case(name, kind, S, C, T, H, **kw):
        return dict(name=name, kind=kind, S=S, C=C, T=T, H=H, **kw)
    return [
        # the smallest pipeline: a first try or a health check; launches and host calls count
        case("step_tiny", "step", 4, 8, 16, 256, dist="gauss", mode="element", tamper="add",
             level=0.05, sigma=1e-3),
        # the paper's own shape, one attack of its Table 1 with every detector setting
        case("table1_paper", "table1", 12, 100, 48, 768, tamper="add", level=0.05, sigma=0.002),
        # the paper's depth / position / collusion substudies, two colluders
        case("chain_paper", "chain", 12, 100, 48, 768, mal=2, carry=0.7, level=0.05, sigma=0.002,
             dist="gauss"),
        # a verifier of a 7B-shaped pipeline scores one delivery of its peers' activations
        case("score_7b", "score", 8, 64, 128, 4096),
        # the same for a 70B-shaped pipeline: the detector's largest call
        case("score_70b", "score", 16, 256, 256, 8192),
        # the 70B-shaped study, three attacks over one reference set (a 128-canary slice)
        case("step_70b", "batch", 16, 128, 256, 8192, runs=3, dist="gauss", mode="element",
             sigma=1e-3),
        # one reference set of the 216-configuration factorial with its 24 runs
        case("sweep_set", "batch", 16, 32, 64, 4096, runs=24, dist="gauss", mode="element",
             sigma=1e-3),
        # heavy-tailed benign noise, a point of the signal-to-noise curve
        case("step_snr_t3", "step", 16, 128, 128, 4096, dist="t3", mode="element", tamper="add",
             level=0.02, sigma=0.01),
        # the simulation study's fast path on the factorial's largest shape
        case("fused_sweep", "fused", 32, 32, 64, 8192, dist="gauss", mode="element",
             tamper="mixed", level=0.02, sigma=1e-3),
        # ranking all of the factorial's 216 configurations
        case("rank_sweep", "rank", 32, 32, 0, 0, configs=216),
        # the offline pass for a 7B-shaped pipeline
        case("refs_7b", "refs", 8, 64, 128, 4096),
        # the metric ablations on a shape that no tile size divides
        case("ablate_ragged", "ablate", 10, 75, 97, 1288),
    ]


#: most elements of a drawn case, by kind: no more work than the largest listed case has
MOST = {"step": 1 << 30, "batch": 3 << 29, "score": 1 << 33, "ablate": 1 << 29, "table1": 1 << 27,
        "chain": 1 << 28, "fused": 1 << 30, "refs": 1 << 29}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, most):
    """S, C, T, H over the ranges in use, the number of elements spread over its logarithm."""
    target = math.exp(rng.uniform(math.log(1 << 17), math.log(most)))
    while True:
        S, C, T = _log_int(rng, 2, 32), _log_int(rng, 8, 256), _log_int(rng, 16, 256)
        H = 8 * _log_int(rng, 32, 1024)
        if target / 3 <= S * C * T * H <= min(3 * target, most):
            return dict(S=S, C=C, T=T, H=H)


def draw(rng):
    kind = rng.choice(["step", "step", "batch", "batch", "score", "score", "ablate", "table1",
                       "chain", "fused", "rank", "refs"])
    if kind == "rank":
        S = _log_int(rng, 3, 64)
        return dict(kind=kind, S=S, C=min(_log_int(rng, 8, 256), 16384 // S), T=0, H=0,
                    configs=_log_int(rng, 1, 216))
    case = dict(kind=kind, **_shape(rng, MOST[kind]))
    if kind in ("step", "batch", "fused", "chain"):
        case["dist"] = rng.choice(["gauss", "gauss", "t3"])
    if kind in ("step", "batch", "fused"):
        case["mode"] = rng.choice(["element", "element", "block"])
    if kind in ("step", "fused", "table1"):
        case["tamper"] = rng.choice(sorted(TAMPERS))
    if kind in ("step", "fused", "table1", "chain"):
        case["level"] = rng.choice([0.005, 0.02, 0.05, 0.1])
    if kind in ("step", "batch", "fused", "table1", "chain"):
        case["sigma"] = rng.choice([1e-4, 1e-3, 2e-3, 1e-2])
    if kind == "chain":
        case.update(carry=rng.choice([0.3, 0.7, 1.0]), mal=rng.randint(1, min(4, case["S"] - 1)))
    if kind == "batch":
        most = max(1, (3 << 31) // (case["S"] * case["C"] * case["T"] * case["H"]))
        case["runs"] = rng.randint(1, min(24, most))
    return case


# -- inputs ------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _refs(case, g):
    """References ~ N(0, 1) with 1% of the channels 20 times larger, a shard at a time."""
    S, C, T, H = (case[k] for k in "SCTH")
    ref = torch.empty((S, C, T, H), dtype=torch.float32, device=DEV)
    big = torch.randperm(H, generator=g, device=DEV)[:max(1, H // 100)]
    gain = torch.ones(H, device=DEV).index_fill_(0, big, 20.0)
    for s in range(S):
        ref[s].normal_(generator=g).mul_(gain)
    return ref


def _delivered(ref, g, sigma=1e-3):
    """fp16 activations near ref, shard S // 2 further off than the others."""
    h = torch.empty(ref.shape, dtype=torch.float16, device=DEV)
    for s in range(ref.shape[0]):
        rel = 0.05 if s == ref.shape[0] // 2 else sigma
        for c in range(0, ref.shape[1], 64):
            a = ref[s, c:c + 64]
            h[s, c:c + 64] = torch.randn(a.shape, generator=g, device=DEV).mul_(rel).add_(1).mul_(a)
    return h


def _stats(ref):
    """rms and mean |a| of each block, [S][C] fp64."""
    sq, ab = [], []
    for a in ref:
        sq.append(torch.stack([x.double().square().mean().sqrt() for x in a]))
        ab.append(torch.stack([x.double().abs().mean() for x in a]))
    return torch.stack(sq), torch.stack(ab)


def _mal(case):
    """The middle shard, or `mal` colluders spaced evenly."""
    c, S = case.get("mal", 1), case["S"]
    return sum(1 << s for s in {min(S - 1, max(0, S * (j + 1) // (c + 1) - 1)) for j in range(c)})


def _run_kw(case, seed, cfg_id, tamper, level, tscale, bscale):
    kw = dict(seed=seed, cfg_id=cfg_id, mal_mask=_mal(case), sigma_b=case["sigma"],
              benign_dist=cdt.DIST_T3 if case.get("dist") == "t3" else cdt.DIST_GAUSS,
              benign_mode=cdt.NOISE_BLOCK if bscale is not None else cdt.NOISE_ELEMENTWISE,
              tamper=TAMPERS[tamper], tscale=tscale, bscale=bscale)
    if tamper in ("flip", "mixed"):
        kw["flip_p"] = level
    if tamper in ("scale", "mixed"):
        kw["scale"] = 1.0 + level
    return kw


def _runs(case):
    """The (tamper, level) of each run of a batch: every attack in turn."""
    names = ["add", "flip", "scale", "mixed"]
    return [(names[r % 4], (0.05, 0.005, 0.02, 0.1)[r // 4 % 4]) for r in range(case["runs"])]


def prepare(case, seed):
    kind, g = case["kind"], _gen(seed)
    st = dict(case=case, kind=kind, seed=seed, ids=1 + seed % 1000)
    if kind == "rank":
        tables = _rank_tables(case)
        n = sum(S * C for S, C, _, _, _ in tables)
        x = torch.rand(n, generator=g, device=DEV).mul_(0.2).add_(0.9)
        noise = torch.empty(n, device=DEV).fill_(1e-3).mul_(x)
        for S, C, off, mask, _ in tables:  # malicious columns shifted, some runs more than others
            mal = torch.tensor([(mask >> s) & 1 for s in range(S)], device=DEV, dtype=torch.bool)
            noise[off:off + S * C].view(C, S)[:, mal] *= 1.0 + 0.1 * ((off // 8) % 4)
        st.update(scores=noise, cfgs=tables, n=len(tables))
        st["table"], _ = cdt.auroc_upload(tables, n, flags=RANK_ALL, like=noise)
        return st
    S, C, T, H = (case[k] for k in "SCTH")
    if kind == "refs":
        return st
    ref = st["ref"] = _refs(case, g)
    if kind in ("score", "ablate"):
        st["h"] = _delivered(ref, g)
        if kind == "ablate":
            st["r"] = _delivered(ref, g)
        st["ws"] = cdt.workspace(S, C, T, H, ref)
        return st
    rms, mu = _stats(ref)
    block = kind in ("table1", "chain") or case["mode"] == "block"
    bscale = st["bscale"] = (case["sigma"] * mu).float() if block else None
    st["ws"] = cdt.workspace(S, C, T, H, ref)
    if kind == "batch":
        runs = _runs(case)
        st["hs"] = [torch.empty(ref.shape, dtype=torch.float16, device=DEV) for _ in runs]
        st["scores"] = torch.empty((len(runs), C, S), device=DEV)
        st["kws"] = [_run_kw(case, seed, st["ids"] + r, tamper, level,
                             (level * rms).float() if TAMPERS[tamper] & cdt.T_ADD else None,
                             bscale) for r, (tamper, level) in enumerate(runs)]
        st["sim"] = cdt.sim_batch([(ref, h, kw) for h, kw in zip(st["hs"], st["kws"])])
        st["drift"] = cdt.drift_batch([(h, ref, sc, None) for h, sc in zip(st["hs"], st["scores"])])
        st["cfgs"] = [(S, C, r * S * C, _mal(case), st["ids"] + r) for r in range(len(runs))]
        st["table"], st["n"] = cdt.auroc_upload(st["cfgs"], st["scores"].numel(), flags=RANK_ALL,
                                                like=ref)
        return st
    st["h"] = torch.empty(ref.shape, dtype=torch.float16, device=DEV)
    tamper = case.get("tamper", "add")
    tscale = None
    if kind in ("step", "fused") and TAMPERS[tamper] & cdt.T_ADD:
        tscale = (case["level"] * rms).float()
    kw = st["kw"] = _run_kw(case, seed, st["ids"], tamper, case["level"], tscale, bscale)
    if kind == "chain":
        kw["carry"] = case["carry"]
    if kind == "table1":
        st["r"] = torch.empty_like(st["h"])
        st["scores"] = torch.empty((4, C, S), device=DEV)
        st["cfgs"] = [(S, C, m * S * C, _mal(case), st["ids"]) for m in range(4)]
        st["kw_redraw"] = dict(kw, mal_mask=0, redraw=True)
    else:
        st["score"] = torch.empty((C, S), device=DEV)
        st["cfgs"] = [(S, C, 0, _mal(case), st["ids"])]
    return st


def _rank_tables(case):
    tables, off, S, C = [], 0, case["S"], case["C"]
    for k in range(case["configs"]):
        s = max(2, S >> (2 - 3 * k // case["configs"]))  # a quarter, a half and all of the shards
        tables.append((s, C, off, 1 << (s // 2), k))
        off += s * C
    return tables


# -- one pass ----------------------------------------------------------------------------

def run(st):
    return globals()["_run_" + st["kind"]](st)


def _ranked(st, scores):
    """Counts of the detector, its controls and the pooled ranking, and Eq. 6 from them."""
    counts, pooled, base = cdt.auroc(st["cfgs"], scores, seed=st["seed"], flags=RANK_ALL)
    return dict(counts=counts, pooled=pooled, base=base,
                values=cdt.auroc_values(counts, pooled, base))


def _run_step(st):
    h = cdt.canary_sim(st["ref"], out=st["h"], **st["kw"])
    score = cdt.drift_score(h, st["ref"], out=st["score"], ws=st["ws"])
    return dict(_ranked(st, score), h=h, score=score)


def _run_batch(st):
    cdt.canary_sim_batch(st["sim"])
    cdt.drift_score_batch(st["drift"])
    counts, pooled, base = cdt.auroc_launch(st["table"], st["n"], st["scores"], seed=st["seed"],
                                            flags=RANK_ALL)
    values = cdt.auroc_values(counts, pooled, base)
    return dict(hs=st["hs"], scores=st["scores"], counts=counts, pooled=pooled, base=base,
                values=values)


def _run_score(st):
    return cdt.drift_score(st["h"], st["ref"], ws=st["ws"])


def _run_ablate(st):
    h, r, ref, ws = st["h"], st["r"], st["ref"], st["ws"]
    return (cdt.drift_score_f16ref(h, r, ws=ws), cdt.cosine_score(h, ref, ws=ws),
            cdt.cosine_score_f16ref(h, r, ws=ws))


def _exact_scale(st):
    kw = {k: v for k, v in st["kw"].items() if k != "tscale"}
    return cdt.tamper_scale_exact(st["ref"], st["case"]["level"], ws=st["ws"], **kw)


def _run_table1(st):
    ref, sc, ws, kw = st["ref"], st["scores"], st["ws"], st["kw"]
    if kw["tamper"] & cdt.T_ADD:
        kw = dict(kw, tscale=_exact_scale(st))
    h = cdt.canary_sim(ref, out=st["h"], **kw)
    r = cdt.canary_sim(ref, out=st["r"], **st["kw_redraw"])
    cdt.drift_score(h, ref, out=sc[0], ws=ws)
    cdt.drift_score_f16ref(h, r, out=sc[1], ws=ws)
    cdt.cosine_score(h, ref, out=sc[2], ws=ws)
    cdt.cosine_score_f16ref(h, r, out=sc[3], ws=ws)
    return dict(_ranked(st, sc), h=h, r=r, scores=sc, tscale=kw["tscale"])


def _run_chain(st):
    tscale = _exact_scale(st)
    h = cdt.canary_sim(st["ref"], out=st["h"], **dict(st["kw"], tscale=tscale))
    score = cdt.drift_score(h, st["ref"], out=st["score"], ws=st["ws"])
    return dict(_ranked(st, score), h=h, score=score, tscale=tscale)


def _run_fused(st):
    return cdt.sim_score(st["ref"], out=st["score"], ws=st["ws"], **st["kw"])


def _run_rank(st):
    counts, pooled, base = cdt.auroc_launch(st["table"], st["n"], st["scores"], seed=st["seed"],
                                            flags=RANK_ALL)
    values = cdt.auroc_values(counts, pooled, base)
    canaries = cdt.auroc_canaries(st["cfgs"], st["scores"], seed=st["seed"])
    return dict(counts=counts, pooled=pooled, base=base, values=values, canaries=canaries)


def _run_refs(st):
    S, C, T, H = (st["case"][k] for k in "SCTH")
    gain = cdt.outlier_gain(H, int(0.01 * H + 0.5), 20.0, st["seed"], st["ids"])
    ref = cdt.ref_synth(S, C, T, H, st["seed"], st["ids"], gain)
    sumsq, sumabs = cdt.ref_stats(ref)
    tscale, bscale = cdt.block_scales(sumsq, sumabs, T, H, 0.05, 1e-3)
    return dict(gain=gain, ref=ref, sumsq=sumsq, sumabs=sumabs, tscale=tscale, bscale=bscale)


# -- what a pass cannot do without ---------------------------------------------------------

def work(case):
    S, C, n = case["S"], case["C"], case["S"] * case["C"] * case["T"] * case["H"]
    # bytes of references, activations and scores, each read or written once
    per = {"step": 6, "score": 6, "ablate": 8, "table1": 8, "chain": 6, "fused": 4, "refs": 4}
    if case["kind"] == "rank":
        tables = _rank_tables(case)
        return dict(bytes=sum(4 * s * c + 160 + 24 * c for s, c, *_ in tables), flops=0)
    if case["kind"] == "batch":
        return dict(bytes=n * (4 + 2 * case["runs"]) + case["runs"] * 4 * S * C, flops=0)
    return dict(bytes=n * per[case["kind"]] + 4 * S * C, flops=0)


def tolerance(case):
    # Activations, references and counts are the same bits whatever the order of the sums; the
    # scores are fp32 roundings of fp64 sums, so two orders differ by one fp32 step at most
    # (1.2e-7 of a value).  A single fp16 activation off by its last bit shows in "max".
    if case["kind"] == "rank":
        return "exact"
    return {"rel": 2e-7, "max": 5e-7, "differ": 0.0}


# -- the same from the definitions, in 64 bits ---------------------------------------------

U32 = 0xFFFFFFFF
STREAM = dict(ref=0, benign=1, t12=2, t3=3, add=4, flip=5, scramble=6, random=7, outlier=8, alt=9)


def _philox(q, c, s, tag, seed):
    """Philox4x32-10 of counter (q, c, s, tag), each an int64 tensor or a number."""
    x, y, z, w = torch.broadcast_tensors(*(torch.as_tensor(v, dtype=torch.int64, device=DEV)
                                           for v in (q, c, s, tag)))
    k0, k1 = seed & U32, (seed >> 32) & U32
    for _ in range(10):
        p0, p1 = x * 0xD2511F53, z * 0xCD9E8D57
        x, y, z, w = (((p1 >> 32) & U32) ^ y ^ k0, p1 & U32, ((p0 >> 32) & U32) ^ w ^ k1, p0 & U32)
        k0, k1 = (k0 + 0x9E3779B9) & U32, (k1 + 0xBB67AE85) & U32
    return x, y, z, w


def _r32(x):
    """fp64 rounded once to fp32."""
    return x.float().double()


UNIT = float(np.float32(math.sqrt(3.0 / (2.0 ** 32 - 1))))


def _irwin_hall(a, b):
    n = (a & 0xFFFF) + (a >> 16) + (b & 0xFFFF) + (b >> 16) - 131070
    return _r32(n.double() * UNIT)


def _normals(n, c, s, tag, seed):
    """n unit normals for each canary in c, one shard and stream: [C][n]."""
    x, y, z, w = _philox(torch.arange(n // 2, device=DEV)[None], c[:, None], s, tag, seed)
    return torch.stack((_irwin_hall(x, y), _irwin_hall(z, w)), -1).view(len(c), n)


def _tag(stream, cfg_id):
    return STREAM[stream] << 24 | cfg_id


def _benign(kw, a, u, s, c, bscale):
    """Eq. 2 on [C][n] fp64: u plus the benign noise of reference a."""
    n, seed, redraw = a.shape[1], kw["seed"], 8 if kw.get("redraw") else 0
    z = _normals(n, c, s, (1 + redraw) << 24 | kw["cfg_id"], seed)
    if kw["benign_dist"] == cdt.DIST_T3:
        x, y, zz, w = _philox(torch.arange(n, device=DEV)[None], c[:, None], s,
                              (2 + redraw) << 24 | kw["cfg_id"], seed)
        z1, z2 = _irwin_hall(x, y), _irwin_hall(zz, w)
        del x, y, zz, w
        z3 = _normals(n, c, s, (3 + redraw) << 24 | kw["cfg_id"], seed)
        q = _r32(_r32(_r32(z1 * z1) + _r32(z2 * z2)) + _r32(z3 * z3))
        z = torch.where(q == 0, 0.0, _r32(z / _r32(q.sqrt())))
    sc = _r32(float(np.float32(kw["sigma_b"])) * a.abs()) if bscale is None else bscale
    return _r32(u + _r32(sc * z))


def _tampered(kw, v, s, c, tscale):
    """Eq. 3 on a malicious shard's [C][n]."""
    n = v.shape[1]
    if kw["tamper"] & cdt.T_ADD:
        v = _r32(v + _r32(tscale * _normals(n, c, s, _tag("add", kw["cfg_id"]), kw["seed"])))
    if kw["tamper"] & cdt.T_FLIP:
        u = _philox(torch.arange(-(-n // 4), device=DEV)[None], c[:, None], s,
                    _tag("flip", kw["cfg_id"]), kw["seed"])
        u = torch.stack(u, -1).view(len(c), -1)[:, :n]
        v = torch.where(u < math.floor(kw["flip_p"] * 2.0 ** 32), -v, v)
    if kw["tamper"] & cdt.T_SCALE:
        v = _r32(float(np.float32(kw["scale"])) * v)
    return v


def _live(ref, kw, tscale=None, eps=None):
    """h of one run, and the exact-norm scales [S][C] where eps is given (else tscale's)."""
    S, C, T, H = ref.shape
    h = torch.empty(ref.shape, dtype=torch.float16, device=DEV)
    ts = torch.zeros((S, C), device=DEV) if tscale is None else tscale.clone()
    carry = float(np.float32(kw.get("carry", 0.0)))
    step = max(1, (1 << 26) // (T * H))
    for c0 in range(0, C, step):
        c = torch.arange(c0, min(C, c0 + step), device=DEV)
        d = None
        for s in range(S):
            a = ref[s, c].double().view(len(c), -1)
            u = a if d is None else _r32(a + _r32(carry * d))
            bs = None if kw["bscale"] is None else kw["bscale"][s, c].double()[:, None]
            v = _benign(kw, a, u, s, c, bs)
            mal = (kw["mal_mask"] >> s) & 1
            if eps is not None and (mal or not carry):
                N = _normals(a.shape[1], c, s, _tag("add", kw["cfg_id"]), kw["seed"])
                ts[s, c] = (eps * (v.square().sum(1) / N.square().sum(1)).sqrt()).float()
            if mal:
                v = _tampered(kw, v, s, c, ts[s, c].double()[:, None])
            out = v.float().half()
            h[s, c] = out.view(len(c), T, H)
            d = _r32(out.double() - a) if carry else None
    return h, ts


def _scores(h, ref, cosine=False):
    """Eq. 4 (or 1 - cos) of every block, [C][S] fp64."""
    out = torch.empty((ref.shape[1], ref.shape[0]), dtype=torch.float64, device=DEV)
    for s in range(ref.shape[0]):
        for c0 in range(0, ref.shape[1], 32):
            a = ref[s, c0:c0 + 32].double().flatten(1)
            d = h[s, c0:c0 + 32].double().flatten(1) - a
            D, A = d.square().sum(1), a.square().sum(1)
            if cosine:
                P = (a * d).sum(1)
                g = (A * (A + 2 * P + D)).sqrt()
                out[c0:c0 + 32, s] = (A * D - P * P) / (g * (g + A + P))
            else:
                out[c0:c0 + 32, s] = (D / A).sqrt()
    return out


def _values(cfgs, scores, seed):
    """Eq. 6, strict and Mann-Whitney, of the detector, control, pooled ranking and baseline."""
    rows = []
    for S, C, off, mask, cid in cfgs:
        m = scores.reshape(-1)[off:off + S * C].view(C, S).double()
        pos = torch.tensor([bool(mask >> s & 1) for s in range(S)], device=DEV)
        t, shard = torch.arange(C, device=DEV), torch.arange(S, device=DEV)
        benign = shard[~pos]
        js = benign[_philox(t, 0, 0, _tag("scramble", cid), seed)[0] % len(benign)]
        u = (_philox(t[:, None], shard[None], 0, _tag("random", cid), seed)[0] >> 8).double()
        row = []

        def ratio(a, b, keep=None):
            keep = torch.ones_like(a > b) if keep is None else keep
            G, E, n = (int(k.sum()) for k in ((a > b) & keep, (a == b) & keep, keep))
            row.extend([G / n, (G + 0.5 * E) / n] if n else [math.nan, math.nan])

        ratio(m[:, pos, None], m[:, None, ~pos])
        ratio(m.gather(1, js[:, None]), m[:, benign], benign[None] != js[:, None])
        ratio(m[:, pos].reshape(-1, 1), m[:, ~pos].reshape(1, -1))
        ratio(u[:, pos, None], u[:, None, ~pos])
        rows.append(row)
    return torch.tensor(rows, dtype=torch.float64, device=DEV)


def exact(case, seed):
    st, kind = prepare(case, seed), case["kind"]
    none = dict(counts=None, pooled=None, base=None)
    if kind == "rank":
        return dict(none, canaries=None, values=_values(st["cfgs"], st["scores"], seed))
    if kind == "refs":
        return _exact_refs(case, seed, st["ids"])
    ref = st["ref"]
    if kind == "score":
        return _scores(st["h"], ref)
    if kind == "ablate":
        h, r = st["h"], st["r"]
        return _scores(h, r), _scores(h, ref, True), _scores(h, r, True)
    if kind == "batch":
        for h, kw in zip(st["hs"], st["kws"]):
            h.copy_(_live(ref, kw, kw["tscale"])[0])
        scores = torch.stack([_scores(h, ref) for h in st["hs"]])
        return dict(none, hs=st["hs"], scores=scores,
                    values=_values(st["cfgs"], scores.float(), seed))
    kw = st["kw"]
    eps = case["level"] if kind == "chain" or (kind == "table1" and kw["tamper"] & 1) else None
    h, ts = _live(ref, kw, kw["tscale"], eps)
    score = _scores(h, ref)
    if kind == "fused":
        return score
    if kind == "table1":
        r = _live(ref, st["kw_redraw"])[0]
        scores = torch.stack([score, _scores(h, r), _scores(h, ref, True), _scores(h, r, True)])
        return dict(none, h=h, r=r, scores=scores, tscale=None if eps is None else ts,
                    values=_values(st["cfgs"], scores.float(), seed))
    out = dict(none, h=h, score=score, values=_values(st["cfgs"], score.float(), seed))
    return dict(out, tscale=ts) if kind == "chain" else out


def _exact_refs(case, seed, rid):
    S, C, T, H = (case[k] for k in "SCTH")
    j = torch.arange(H, device=DEV)
    w = _philox(j, 0, 0, _tag("outlier", rid), seed)[0]
    gain = torch.ones(H, dtype=torch.float64, device=DEV)
    gain[torch.argsort(w * 65536 + j)[:int(0.01 * H + 0.5)]] = 20.0
    ref = torch.empty((S, C, T, H), device=DEV)
    for s in range(S):
        for c0 in range(0, C, 16):
            c = torch.arange(c0, min(C, c0 + 16), device=DEV)
            z = _normals(T * H, c, s, _tag("ref", rid), seed).view(len(c), T, H)
            ref[s, c] = (z * gain).float()
    sumsq = torch.stack([a.double().square().sum((1, 2)) for a in ref])
    sumabs = torch.stack([a.double().abs().sum((1, 2)) for a in ref])
    return dict(gain=gain, ref=ref, sumsq=sumsq, sumabs=sumabs,
                tscale=0.05 * (sumsq / (T * H)).sqrt(), bscale=1e-3 * (sumabs / (T * H)))
