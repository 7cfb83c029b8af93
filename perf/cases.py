"""Performance cases of the CertKV compression pass and of decode over its cache.

A case names one public entry point (or the few that a program calls one
after the other) and the shape of its cache:

  compress   the whole pass: score, order, curves, allocation, selection, tail
             slot and packed cache, into preallocated outputs
  staged     the stages one by one for a program with scores of its own:
             order, curves and budgets, kept sets, tail summary, packed cache
  coverage   coverage budgets and kept masks from a program's own scores
  decode     tq new queries per sequence over a packed cache
  clusters   clustered tail summaries of the evicted ranks
  certified  decode over kept rows and cluster summaries, with the certificate

Shapes are those of the repository's own workloads (Llama-3-8B and 70B class
caches, a tiny fp32 cache, ragged batches) and generic ones around them.
Inputs are synthetic: normal keys and queries, planted keys on half of the
heads, Student-t or normal values scaled per head.
"""
import math

import torch

import paper_2608_21541_amd as ck

DEV = "cuda:0"


def _case(name, kind, layers, seqlens, heads=8, group=4, dim=128, window=64, dtype="bf16",
          keep=0.10, tail="t3", lse=False, tq=0, m=0, retain=0.9):
    c = dict(kind=kind, layers=layers, seqlens=",".join(str(n) for n in seqlens), heads=heads,
             group=group, dim=dim, window=window, dtype=dtype, keep=keep, values=tail,
             lse_in=lse, tq=tq, clusters=m, retain=retain)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The tiny fp32 cache without grouping: latency and launches.
        _case("compress_tiny_f32", "compress", 1, [1024], heads=4, group=1, dim=64, window=16,
              dtype="f32", keep=0.125, tail="gauss"),
        # One layer of an 8B-class model at 32K: a program that compresses each
        # layer as its prefill ends makes one such call per layer.
        _case("compress_layer_32k", "compress", 1, [32768], tail="gauss"),
        # A ragged batch of eight prompts, one layer, 20-fold budget.
        _case("compress_ragged_8", "compress", 1,
              [58321, 8192, 41007, 20480, 12345, 65536, 30011, 15873], window=32, keep=0.05,
              tail="gauss"),
        # Four layers of a 70B-class model (512 window rows per KV head) at an
        # odd length, the prefill's row log-sum-exp handed over.
        _case("compress_70b_4l_lse", "compress", 4, [49157], group=8, keep=0.05, lse=True),
        # The whole 8B-class cache at 128K: the repository's headline workload.
        _case("compress_8b_32l_128k", "compress", 32, [131072]),
        # A scorer of the caller's own, stage by stage: two prompts, one layer.
        _case("staged_2seq", "staged", 1, [65537, 24001]),
        # Coverage budgets at 90 % retained mass, a small batch, two layers.
        _case("coverage_3seq", "coverage", 2, [16384, 9999, 30001]),
        # One new token over one layer's packed cache: the layer-by-layer step
        # of a decoding model.
        _case("decode_layer_tq1", "decode", 1, [32768], tq=1),
        # One new token over every layer of the 8B-class cache.
        _case("decode_8b_32l_tq1", "decode", 32, [131072], tq=1),
        # A block of 32 new queries (speculative or chunked continuation).
        _case("decode_8b_32l_tq32", "decode", 32, [131072], tq=32),
        # Sixteen summaries per head over four layers' evicted ranks.
        _case("clusters_4l_32k", "clusters", 4, [32768], m=16),
        # Certified decode of a small batch, two layers.
        _case("certified_2l_tq4", "certified", 2, [32768, 11111], tq=4, m=16),
    ]


MOST_TOKENS = 12 * 131072  # layers x tokens of a drawn case at 8 heads of 128


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["compress", "compress", "compress", "staged", "coverage", "decode",
                       "decode", "clusters", "certified"])
    f32 = kind in ("compress", "staged", "clusters") and rng.random() < 0.2
    dim = 64 if f32 else rng.choice([64, 128, 128])  # fp32 caches have rows of 64
    heads = rng.choice([4, 8, 8, 16]) if not f32 else rng.choice([4, 8])
    group = rng.choice([1, 4, 4]) if f32 else rng.choice([1, 4, 4, 8])
    window = rng.choice([16, 32, 64, 64])
    batch = rng.choice([1, 1, 2, 3, 8])
    most = 16384 if f32 else 131072
    seqlens = [_log_int(rng, 1024, most) for _ in range(batch)]
    if rng.random() < 0.3:  # whole multiples are common too
        seqlens = [max(1024, n // 1024 * 1024) for n in seqlens]
    cap = MOST_TOKENS * 8 * 128 // (heads * dim) // (8 if f32 else 1)
    layers = min(_log_int(rng, 1, 32), max(1, cap // sum(seqlens)))
    return _case(None, kind, layers, seqlens, heads=heads, group=group, dim=dim, window=window,
                 dtype="f32" if f32 else "bf16", keep=rng.choice([0.05, 0.1, 0.2]),
                 tail=rng.choice(["t3", "gauss"]),
                 lse=kind == "compress" and rng.random() < 0.25,
                 tq=rng.choice([1, 1, 2, 8, 32]) if kind in ("decode", "certified") else 0,
                 m=rng.choice([4, 16, 64]) if kind in ("clusters", "certified") else 0,
                 retain=rng.choice([0.8, 0.9, 0.95]))


def _lens(case):
    return [int(n) for n in case["seqlens"].split(",")]


def _n_keep(case):
    return [int(math.floor(case["keep"] * n)) + 1 for n in _lens(case)]


def _spec(case):
    clustered = case["kind"] in ("clusters", "certified")
    return ck.ProblemSpec(case["layers"], case["heads"], case["group"], case["dim"],
                          case["window"], _lens(case),
                          torch.float32 if case["dtype"] == "f32" else torch.bfloat16,
                          slot=not clustered)


def _values(case, gen, n):
    H, d = case["heads"], case["dim"]
    v = torch.randn((n, H, d), generator=gen, device=DEV)
    if case["values"] == "t3":
        chi = torch.randn((n, H, 3), generator=gen, device=DEV).square_().sum(-1, keepdim=True)
        v *= torch.rsqrt(chi / 3.0)
    lo, hi = math.log(0.2), math.log(5.0)
    return v.mul_(torch.exp(lo + (hi - lo) * torch.rand((1, H, 1), generator=gen, device=DEV)))


def _cache(case, gen):
    """Window queries, keys and values; half of the heads hold 16 planted keys."""
    L, H, G, d, w = (case[x] for x in ("layers", "heads", "group", "dim", "window"))
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    lens = _lens(case)
    T, B = sum(lens), len(lens)
    q = torch.randn((L, B * w, H * G, d), generator=gen, device=DEV).to(dt)
    k = torch.empty((L, T, H, d), dtype=dt, device=DEV)
    v = torch.empty_like(k)
    for l in range(L):
        t0 = 0
        for b, n in enumerate(lens):
            kk = torch.randn((n, H, d), generator=gen, device=DEV)
            v[l, t0:t0 + n] = _values(case, gen, n)
            qb = q[l, b * w:(b + 1) * w].float().view(w, H, G, d).mean((0, 2))[: H // 2]
            lift = 5.0 * math.sqrt(d) * qb / qb.square().sum(-1, keepdim=True)
            pos = torch.randint(0, n - w, (16,), generator=gen, device=DEV)
            kk[pos, : H // 2] += lift
            k[l, t0:t0 + n] = kk
            t0 += n
    return q, k, v


def _scores(case, gen):
    """Window masses of a scorer: log-normal, a few large ones on half of the heads."""
    L, H, T = case["layers"], case["heads"], sum(_lens(case))
    s = torch.exp(0.35 * torch.randn((L, H, T), generator=gen, device=DEV))
    few = torch.rand((L, H // 2, T), generator=gen, device=DEV) < 16.0 / T
    s[:, : H // 2] *= torch.where(few, 150.0, 1.0)
    t0 = 0
    for n in _lens(case):
        s[..., t0:t0 + n] *= case["window"] * case["group"] / n
        t0 += n
    return s


def _budgets(case, gen):
    """Budgets [L][B][H] of an uneven allocation: each (layer, sequence) sums to H (n_keep - 1)."""
    L, H = case["layers"], case["heads"]
    out = []
    for n, nk in zip(_lens(case), _n_keep(case)):
        real = H * (nk - 1)
        floor = max(1, int(0.2 * real / H))
        share = torch.exp(1.2 * torch.randn((L, H), generator=gen, device=DEV).double())
        share /= share.sum(-1, keepdim=True)
        b = floor + (share * (real - H * floor)).long()
        b.clamp_(max=n - 1)
        out.append(b)
    return torch.stack(out, 1)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 1000003 + 17)
    spec, kind = _spec(case), case["kind"]
    L, H, G, d, T = case["layers"], case["heads"], case["group"], case["dim"], sum(_lens(case))
    st = dict(case=case, spec=spec)
    if kind == "compress":
        st["q"], st["k"], st["v"] = _cache(case, gen)
        st["n_keep"] = _n_keep(case)
        st["lse_in"] = _window_lse(case, st["q"], st["k"]) if case["lse_in"] else None
        st["bufs"] = ck.CompressBuffers(spec, st["n_keep"], torch.device(DEV))
    elif kind == "coverage":
        st["scores"] = _scores(case, gen)
    elif kind in ("staged", "clusters"):
        _, st["k"], st["v"] = _cache(case, gen)
        st["scores"] = _scores(case, gen)
        st["n_keep"] = _n_keep(case)
        if kind == "clusters":
            st["budgets"] = _budgets(case, gen).reshape(-1).int()
            st["perm"] = torch.cat([torch.sort(s, dim=-1, descending=True, stable=True)[1]
                                    for s in st["scores"].split(_lens(case), dim=-1)],
                                   -1).int().contiguous()
    else:
        rows = _budgets(case, gen).reshape(-1) + (1 if spec.slot else 0)
        st["off"] = torch.zeros(rows.numel() + 1, dtype=torch.int64, device=DEV)
        st["off"][1:] = rows.cumsum(0)
        R = int(st["off"][-1])
        st["kp"] = torch.randn((R, d), generator=gen, device=DEV).bfloat16()
        st["vp"] = torch.randn((R, d), generator=gen, device=DEV).bfloat16()
        tq = case["tq"]
        st["qn"] = torch.randn((L, len(_lens(case)) * tq, H * G, d), generator=gen,
                               device=DEV).bfloat16()
        st["max_rows"] = int(rows.max())
        if kind == "decode":
            st["bufs"] = ck.DecodeBuffers(spec, tq, torch.device(DEV), with_lse=True,
                                          max_rows=st["max_rows"])
        else:
            m, U = case["clusters"], spec.units
            r = lambda *s: torch.rand(s, generator=gen, device=DEV)  # noqa: E731
            st["cl"] = dict(
                kbar=(0.1 * torch.randn((U, m, d), generator=gen, device=DEV)).bfloat16(),
                vbar=(0.1 * torch.randn((U, m, d), generator=gen, device=DEV)).bfloat16(),
                count=(1 + 2000 * r(U, m)).int(), rk=0.01 + 0.03 * r(U, m), rv=0.5 + r(U, m),
                vmax_kept=15 + r(U))
    return st


def run(st):
    case, spec, kind = st["case"], st["spec"], st["case"]["kind"]
    if kind == "compress":
        b = ck.compress(spec, st["q"], st["k"], st["v"], st["n_keep"], bufs=st["bufs"],
                        lse_in=st["lse_in"])
        return dict(scores=b.scores, budgets=b.budgets, kept_offsets=b.kept_offsets,
                    kept_idx=b.kept_idx, k_star=b.k_star, v_star=b.v_star, tail_mass=b.tail_mass,
                    k_packed=b.k_packed, v_packed=b.v_packed, pos_packed=b.pos_packed,
                    packed_offsets=b.packed_offsets)
    if kind == "staged":
        a = ck.allocate(spec, st["scores"], st["v"], st["n_keep"], with_perm=True,
                        with_curves=True, with_vsum=True)
        _, off, idx = ck.select(spec, st["scores"], a["budgets"])
        ks, vs, mass = ck.tail_summary(spec, st["scores"], st["k"], st["v"], off, idx)
        kp, vp, pos, po = ck.compact(spec, st["k"], st["v"], off, idx, ks, vs)
        return dict(a, kept_offsets=off, kept_idx=idx, k_star=ks, v_star=vs, tail_mass=mass,
                    k_packed=kp, v_packed=vp, pos_packed=pos, packed_offsets=po)
    if kind == "coverage":
        b, off, _, mask = ck.select(spec, st["scores"], mode="coverage",
                                    retain_mass=case["retain"], with_mask=True)
        return dict(budgets=b, kept_offsets=off, kept_mask=mask)
    if kind == "decode":
        out, lse = ck.decode(spec, st["qn"], st["kp"], st["vp"], st["off"], case["tq"],
                             with_lse=True, bufs=st["bufs"])
        return dict(out=out, lse=lse)
    if kind == "clusters":
        return ck.cluster_tail(spec, st["k"], st["v"], st["perm"], st["budgets"],
                               case["clusters"])
    out, lse, bound = ck.decode_clustered(spec, st["qn"], st["kp"], st["vp"], st["off"],
                                          case["tq"], st["cl"], max_rows=st["max_rows"])
    return dict(out=out, lse=lse, bound=bound)


def work(case):
    L, H, G, d, w = (case[x] for x in ("layers", "heads", "group", "dim", "window"))
    lens, kind = _lens(case), case["kind"]
    e = 4 if case["dtype"] == "f32" else 2
    B, keys = len(lens), L * H * sum(lens)
    units = L * B * H
    kept = L * H * sum(nk - 1 for nk in _n_keep(case))
    cache = 2 * keys * d * e
    if kind == "compress":
        # inputs once; scores, kept positions twice, kept rows and slots out
        return dict(bytes=L * B * w * H * G * d * e + cache + 4 * keys + 8 * kept +
                    2 * (kept + units) * d * e + units * (8 * d + 40),
                    flops=2.0 * keys * w * G * d + 8.0 * keys * d)
    if kind == "staged":  # scores, K, V in; order, curves, kept sets and rows out
        return dict(bytes=cache + 12 * keys + 8 * kept + 2 * (kept + units) * d * e +
                    units * (16 * d + 40), flops=12.0 * keys * d)
    if kind == "coverage":  # scores in, mask and positions out
        return dict(bytes=5 * keys + 4 * case["retain"] * keys, flops=2.0 * keys)
    if kind == "clusters":
        return dict(bytes=cache + 4 * keys + units * case["clusters"] * (2 * d * e + 12),
                    flops=10.0 * keys * d)
    rows, M = kept + (units if kind == "decode" else 0), case["tq"] * G
    extra = units * case["clusters"] * (4 * d + 12)
    return dict(bytes=4 * rows * d + units * M * (6 * d + 8) + extra, flops=4.0 * rows * M * d)


def tolerance(case):
    kind = case["kind"]
    if kind == "compress":
        # Scores are fp32 softmax sums (8e-7 off at most); the slot's keys are
        # small differences of fp32 key sums (1.6e-4 off on the largest case);
        # every whole number follows from the scores' bits.
        return {"rel": 6e-4, "max": 6e-3}
    if kind == "coverage":
        return "exact"
    if kind == "staged":
        # fp64 sums, rounded once to fp32 (3e-8 off); the packed slot's rounding
        # to bf16 may turn over; the whole numbers follow from the curves
        return {"rel": 2e-7, "max": 4e-3}
    if kind == "clusters":
        # fp64 sums rounded to the cache's type (bf16: 2e-3 off on every side),
        # where a rounding may turn over
        return {"rel": 1e-4, "max": 1e-2}
    # fp32 softmax with the weights in two bf16 parts (2.5e-6 off)
    return {"rel": 1e-5, "max": 1e-4}


# ---- the same outputs in 64 bits, in plain torch ------------------------------


def _window_rows(case, q, k, l, b, h):
    """Logits [w*G][n] of one unit in fp64, -inf where masked."""
    lens, G, w = _lens(case), case["group"], case["window"]
    t0, n = sum(lens[:b]), lens[b]
    qh = q[l, b * w:(b + 1) * w, h * G:(h + 1) * G].double().reshape(w * G, -1)
    z = qh @ k[l, t0:t0 + n, h].double().t().contiguous() / math.sqrt(case["dim"])
    row = torch.arange(w * G, device=DEV).unsqueeze(1) // G
    z[:, n - w:].masked_fill_(torch.arange(w, device=DEV) > row, -math.inf)
    return z


def _window_lse(case, q, k):
    """Row log-sum-exp [L][B*w][Hq] fp32, as an attention prefill has it."""
    L, H, G, w, B = case["layers"], case["heads"], case["group"], case["window"], len(_lens(case))
    out = torch.empty((L, B * w, H * G), device=DEV)
    for l in range(L):
        for b in range(B):
            for h in range(H):
                lse = torch.logsumexp(_window_rows(case, q, k, l, b, h), 1)
                out[l, b * w:(b + 1) * w, h * G:(h + 1) * G] = lse.view(w, G)
    return out


def _units(case):
    lens = _lens(case)
    for l in range(case["layers"]):
        for b in range(len(lens)):
            for h in range(case["heads"]):
                yield l, b, h, sum(lens[:b]), sum(lens[:b + 1])


def _order(s):
    return torch.sort(s, descending=True, stable=True)[1]


def exact(case, seed):
    st = prepare(case, seed)
    kind, L, H, G, d = (case[x] for x in ("kind", "layers", "heads", "group", "dim"))
    U = st["spec"].units
    if kind == "compress":
        # What follows the allocation turns on single ranks and has no exact value.
        s = torch.empty((L, H, sum(_lens(case))), dtype=torch.float64, device=DEV)
        for l, b, h, t0, t1 in _units(case):
            z = _window_rows(case, st["q"], st["k"], l, b, h)
            if st["lse_in"] is not None:
                w = case["window"]
                z -= st["lse_in"][l, b * w:(b + 1) * w, h * G:(h + 1) * G].reshape(-1, 1).double()
            else:
                z -= torch.logsumexp(z, 1, keepdim=True)
            s[l, h, t0:t1] = z.exp_().sum(0)
        return dict(scores=s, budgets=None, kept_offsets=None, kept_idx=None, k_star=None,
                    v_star=None, tail_mass=None, k_packed=None, v_packed=None, pos_packed=None,
                    packed_offsets=None)
    if kind == "coverage":
        return None
    if kind == "staged":
        # The slot follows from budgets that turn on single bits of the curves.
        shape = st["scores"].shape
        curves = torch.empty(shape, dtype=torch.float64, device=DEV)
        vsum = torch.empty((U, d), dtype=torch.float64, device=DEV)
        for u, (l, b, h, t0, t1) in enumerate(_units(case)):
            s = st["scores"][l, h, t0:t1].double()
            o = _order(st["scores"][l, h, t0:t1])
            v = st["v"][l, t0:t1, h].double()
            vsum[u] = (s[:, None] * v).sum(0)
            a, v = (s / s.sum())[o].flip(0), v[o].flip(0)
            m, q = a.cumsum(0), (a * v.square().sum(1)).cumsum(0)
            w2 = (a[:, None] * v).cumsum_(0).square_().sum(1)
            curves[l, h, t0:t1] = (m * q - w2).clamp_(min=0).sqrt().flip(0)
        return dict(budgets=None, perm=None, curves=curves, vsum=vsum, kept_offsets=None,
                    kept_idx=None, k_star=None, v_star=None, tail_mass=None, k_packed=None,
                    v_packed=None, pos_packed=None, packed_offsets=None)
    if kind == "clusters":
        m, dt = case["clusters"], st["k"].dtype
        mean = [torch.zeros((U, m, d), dtype=torch.float64, device=DEV) for _ in range(2)]
        rad = [torch.zeros((U, m), dtype=torch.float64, device=DEV) for _ in range(2)]
        vmax = torch.zeros(U, dtype=torch.float64, device=DEV)
        for u, (l, b, h, t0, t1) in enumerate(_units(case)):
            bud = int(st["budgets"][u])
            o = st["perm"][l, h, t0:t1].long()
            x = [y[l, t0:t1, h][o].double() for y in (st["k"], st["v"])]
            vmax[u] = x[1][:bud].norm(dim=1).max()
            size = -(-(t1 - t0 - bud) // m)
            for g in range(m):
                lo, hi = bud + g * size, min(t1 - t0, bud + (g + 1) * size)
                if lo >= hi:
                    continue
                stride = min(16, max(1, (hi - lo) // 64))
                for i in range(2):
                    rows = x[i][lo:hi]
                    mean[i][u, g] = rows.mean(0)
                    stored = rows.mean(0).float().to(dt).double()
                    c = rows[::stride].mean(0)
                    rad[i][u, g] = (rows - c).norm(dim=1).max() + (c - stored).norm()
        return dict(kbar=mean[0], vbar=mean[1], count=None, rk=rad[0], rv=rad[1], vmax_kept=vmax)
    B, tq, scale = len(_lens(case)), case["tq"], 1.0 / math.sqrt(d)
    out = torch.empty((L, B * tq, H * G, d), dtype=torch.float64, device=DEV)
    lse = torch.empty((L, B * tq, H * G), dtype=torch.float64, device=DEV)
    bound = torch.empty_like(lse)
    for u, (l, b, h, _, _) in enumerate(_units(case)):
        r0, r1 = int(st["off"][u]), int(st["off"][u + 1])
        rows, cols = slice(b * tq, (b + 1) * tq), slice(h * G, (h + 1) * G)
        q = st["qn"][l, rows, cols].double().reshape(tq * G, d)
        e = scale * (q @ st["kp"][r0:r1].double().t().contiguous())
        v = st["vp"][r0:r1].double()
        if kind == "certified":
            cl = {k: x[u].double() for k, x in st["cl"].items()}
            lbar = scale * (q @ cl["kbar"].t().contiguous())
            top = torch.maximum(e.amax(1, keepdim=True), lbar.amax(1, keepdim=True))
            we, wc = (e - top).exp(), cl["count"] * (lbar - top).exp()
            z = we.sum(1) + wc.sum(1)
            o = (we @ v + wc @ cl["vbar"]) / z[:, None]
            er = (scale * q.norm(dim=1, keepdim=True) * cl["rk"]).exp()
            zeta, vbar = wc / z[:, None], cl["vbar"].norm(dim=1)
            dz = ((er - 1) * er * zeta).sum(1)
            dn = (er * zeta * ((er - 1) * vbar + cl["rv"])).sum(1)
            vp = torch.maximum(cl["vmax_kept"], (vbar + cl["rv"]).max())
            bound[l, rows, cols] = torch.where(dz <= 1 / 3, 3 * (dn + vp * dz),
                                               math.inf).view(tq, G)
            lse[l, rows, cols] = (z.log() + top[:, 0]).view(tq, G)
        else:
            o = torch.softmax(e, 1) @ v
            lse[l, rows, cols] = torch.logsumexp(e, 1).view(tq, G)
        out[l, rows, cols] = o.view(tq, G, d)
    return dict(out=out, lse=lse, bound=bound) if kind == "certified" else dict(out=out, lse=lse)
