"""Edges of the kernels' size rules: each test runs the sizes at which a
stage changes its split of the work (tiles, remainders, the smallest and the
largest of a range) against the oracle or a plain fp64 reference."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_21541_amd as ck
import synth
from _parity import spec_of

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.init()


def _scores(shape, seed):
    rng = np.random.default_rng(seed)
    return np.exp(rng.standard_normal(shape)).astype(np.float32)


@pytest.mark.parametrize("name,lens", [("C2", [64, 511, 513, 2049, 5000]), ("C1", [16, 700, 4097])])
def test_direct_tail_splits(name, lens):
    # The evicted rows summed directly, split over a unit's slices of
    # positions: slices of part of a list tile and of several, all-zero scores
    # (uniform weights), and scores that leave whole slices without weight.
    # fp64 sums rounded once to fp32: half an ulp plus the sums' own rounding.
    cfg = synth.config(name, seqlens=lens)
    cache = synth.make_cache(cfg, "cpu")
    spec = spec_of(cfg)
    s = _scores((1, cfg.kv_heads, sum(lens)), 3)
    s[0, 0] = 0.0
    s[0, 1, ::3] = 0.0
    s[0, 2, 40:] = 0.0
    st = torch.from_numpy(s).to(DEV)
    k, v = cache["k"].to(DEV), cache["v"].to(DEV)
    bud = torch.tensor([max(1, n // (2 + h)) for n in lens for h in range(cfg.kv_heads)],
                       dtype=torch.int32, device=DEV)
    _, off, idx = ck.select(spec, st, bud)
    ks, vs, mass = ck.tail_summary(spec, st, k, v, off, idx)
    off, idx = off.tolist(), idx.cpu()
    t0 = 0
    for b, n in enumerate(lens):
        for h in range(cfg.kv_heads):
            u = b * cfg.kv_heads + h
            w = torch.from_numpy(s[0, h, t0:t0 + n]).double()
            if w.sum() == 0:
                w = torch.ones(n, dtype=torch.float64)
            tot = w.sum()
            w[idx[off[u]:off[u + 1]].long()] = 0.0
            assert abs(mass[u].item() - (w.sum() / tot).item()) <= 1e-12
            for got, x in ((ks[u], cache["k"]), (vs[u], cache["v"])):
                rows = x[0, t0:t0 + n, h].double()
                ref = (w @ rows) / w.sum() if w.sum() > 0 else torch.zeros(cfg.head_dim).double()
                scale = (w.abs() @ rows.abs()) / max(w.sum().item(), 1e-300)
                assert ((got.cpu().double() - ref).abs() <= 2.0 ** -24 * ref.abs() + 1e-13 * scale).all()
        t0 += n


@pytest.mark.parametrize("n", [16, 63, 64, 65, 1023, 1024, 1025, 16385, 40001])
def test_coverage_budget_sizes(n):
    # Rank ranges narrowed once, twice, not at all; ties with the retained
    # mass (flat and quantized scores, retain = 1), where the serial sums
    # decide; an all-zero head.  Budgets and masks equal the oracle's.
    cfg = synth.config("C1", seqlens=[n], layers=2)
    spec = spec_of(cfg)
    s = _scores((2, 4, n), n)
    s[0, 0] = 0.25
    s[0, 1] = np.round(s[0, 1] * 4) / 4
    s[0, 2] = 0.0
    s[0, 3, 0] = 1e6
    s[1, 0, n // 2:] = 0.0
    s[1, 1] = -s[1, 1]
    s[1, 2, ::5] = -1.0
    st = torch.from_numpy(s).to(DEV)
    for retain in (1e-9, 0.5, 0.9, 0.999, 1.0):
        bud, off, idx, mask = ck.select(spec, st, mode="coverage", retain_mass=retain,
                                        with_mask=True)
        bud, off, idx, mask = bud.cpu(), off.tolist(), idx.cpu().numpy(), mask.cpu().numpy()
        for u in range(8):
            sh = s[u // 4, u % 4]
            perm = oracle.order(sh)
            k = oracle.coverage(sh, perm, retain)
            assert bud[u].item() == k, (retain, u)
            kept = oracle.select(perm, k)
            assert np.array_equal(idx[off[u]:off[u + 1]], kept)
            ref = np.zeros(n, np.uint8)
            ref[kept] = 1
            assert np.array_equal(mask[u // 4, u % 4], ref)


@pytest.mark.parametrize("lens,heads,layers", [
    ([4096], 4, 1),                  # segments of one chunk
    ([5120 + 1], 8, 1),              # one rank in the last chunk
    ([20000, 1024, 513], 8, 1),      # units of forty chunks, two chunks and a rank, and two
    ([40000, 511], 16, 2),           # segments of several chunks beside a unit of one
])
@pytest.mark.parametrize("name", ["C2", "C1"])
def test_curve_segments(name, lens, heads, layers):
    # A unit's curve walk cut into segments: curves, order, value totals and
    # budgets against the oracle's one-piece sums.
    cfg = synth.config(name, seqlens=lens, layers=layers)
    cfg.kv_heads = heads
    cache = synth.make_cache(cfg, "cpu")
    spec = spec_of(cfg)
    s = _scores((layers, heads, sum(lens)), 7)
    s[0, 0] = 0.5                                # flat: every key ties
    s[-1, 1, ::2] = 0.0
    n_keep = [max(2, n // 10) for n in lens]
    al = ck.allocate(spec, torch.from_numpy(s).to(DEV), cache["v"].to(DEV), n_keep,
                     with_perm=True, with_curves=True, with_vsum=True)
    al = {x: y.cpu().numpy() for x, y in al.items()}
    v = cache["v"].double().numpy()
    for l in range(layers):
        t0 = 0
        for b, n in enumerate(lens):
            got = al["curves"][l, :, t0:t0 + n]
            for h in range(heads):
                perm = oracle.order(s[l, h, t0:t0 + n])
                assert np.array_equal(al["perm"][l, h, t0:t0 + n], perm)
                vh = v[l, t0:t0 + n, h]
                c = oracle.curves(s[l, h, t0:t0 + n], perm, vh)[0]
                # (the block checks' bound: fp64 sums in another order)
                tol = 4.0 * np.spacing(c.astype(np.float32)).astype(np.float64) + 1e-6 * c.max()
                assert (np.abs(got[h] - c) <= tol).all()
                u = (l * len(lens) + b) * heads + h
                w = np.maximum(s[l, h, t0:t0 + n], 0).astype(np.float64)
                ref, scale = w @ vh, w @ np.abs(vh)
                assert (np.abs(al["vsum"][u] - ref) <= n * 2.0 ** -51 * scale).all()
            u0 = (l * len(lens) + b) * heads
            ref, _ = oracle.allocate(got, n_keep[b])
            assert np.array_equal(al["budgets"][u0:u0 + heads], ref)
            t0 += n


def _samples(n):
    # Positions that the sort's splitters are chosen from (sort_sample).
    ns = -(-2 * n // 4096) * 32
    i = np.arange(ns, dtype=np.int64)
    lo, hi = i * n // ns, (i + 1) * n // ns
    x = (i * 0x9E3779B1) & 0xFFFFFFFF
    x = ((x ^ x >> 15) * 0x2C1B3C6D) & 0xFFFFFFFF
    x ^= x >> 13
    return lo + (x * (hi - lo) >> 32)


def _largest_bucket(s, perm):
    # Elements between every 32nd sample of a unit in its order `perm`.
    rank = np.empty(len(s), np.int64)
    rank[perm] = np.arange(len(s))
    cut = np.sort(rank[_samples(len(s))])[32::32]
    return np.diff(np.concatenate([[0], cut, [len(s)]])).max()


@pytest.mark.parametrize("lens", [[16], [4095], [4096, 33], [4097, 4096], [8193], [32768, 100, 5000],
                                  [32769], [70001, 33000], [262144], [262145]])
@pytest.mark.parametrize("keep_window", [False, True])
def test_sort_sizes(lens, keep_window):
    # One LDS sort, buckets by value beside units of one, and the edges between
    # them: random scores, ties (flat, quantized, signed zeros), order that
    # follows the position, and every score that is not a sample above all the
    # samples, ties among them, so that the first bucket holds nearly the whole
    # unit, outgrows LDS and is sorted through memory.
    cfg = synth.config("C1", seqlens=lens, layers=2)
    n_all, w = sum(lens), cfg.window
    starts = np.concatenate([[0], np.cumsum(lens)])
    s = _scores((2, 4, n_all), n_all)
    s[0, 1] = 0.5
    s[0, 2] = np.round(s[0, 2] * 2) / 2 - 1.0
    s[0, 2, ::7] = -0.0
    s[0, 3] = np.arange(n_all) / n_all
    s[1, 0] = np.arange(n_all)[::-1] / n_all
    s[1, 1, : n_all // 3] += 1e4
    s[1, 2, ::3] = np.round(s[1, 2, ::3] * 4) / 4
    s[1, 2] += 1e3
    for t0, n in zip(starts, lens):
        s[1, 2, t0 + _samples(n)] -= np.float32(1e3)
    s[1, 3, : n_all // 2] = 0.25                 # one long tie across runs, then spread scores
    spec = spec_of(cfg)
    spec.keep_window = keep_window
    v = torch.zeros((2, n_all, 4, 64), device=DEV)
    if keep_window and min(lens) <= w:
        pytest.skip("the window is the whole sequence: nothing to evict")
    # (a kept window needs b_min = floor(alpha (n_keep - 1)) >= w)
    perm = ck.allocate(spec, torch.from_numpy(s).to(DEV), v, list(lens), alpha=1.0,
                       with_perm=True)["perm"].cpu().numpy()
    for l in range(2):
        for h in range(4):
            for t0, n in zip(starts, lens):
                sh = s[l, h, t0:t0 + n]
                ref = oracle.order(sh, keep_window=w if keep_window else 0)
                assert np.array_equal(perm[l, h, t0:t0 + n], ref), (l, h, n)
                if (l, h) == (1, 2) and n >= 5000:
                    assert _largest_bucket(sh, ref) > 4096


@pytest.mark.parametrize("layers,heads", [(1, 128), (43, 3), (4, 64), (257, 1), (385, 1), (96, 8),
                                          (769, 1)])
@pytest.mark.parametrize("lens", [[8192], [4097], [8193]])
def test_sort_of_many_units(layers, heads, lens):
    # Units of up to 8192 keys sorted by a workgroup each or in buckets, by
    # their number.
    layers, heads = (layers, heads) if heads <= 64 else (layers * heads // 64, 64)
    spec = ck.ProblemSpec(layers, heads, 1, 64, 16, lens, torch.float32)
    s = np.round(_scores((layers, heads, lens[0]), 31) * 256) / 256
    st = torch.from_numpy(s).to(DEV)
    v = torch.zeros((layers, lens[0], heads, 64), device=DEV)
    perm = ck.allocate(spec, st, v, [lens[0] // 10], with_perm=True)["perm"].cpu().numpy()
    for u in {0, 1, layers * heads // 2, layers * heads - 1}:
        l, h = u // heads, u % heads
        assert np.array_equal(perm[l, h], oracle.order(s[l, h])), u


@pytest.mark.parametrize("period", [2, 16, 64, 128])
def test_sort_of_periodic_scores(period):
    # Scores with a period keep the buckets even: within three times the time
    # of scores without one (a bucket of most of a unit takes ten times and more).
    n, units = 65536, 64
    spec = ck.ProblemSpec(units // 8, 8, 1, 64, 16, [n])
    bud = torch.full((units,), n // 10, dtype=torch.int32, device=DEV)
    s = torch.from_numpy(_scores((units // 8, 8, n), 21)).to(DEV)
    p = s + 10.0 * (torch.arange(n, device=DEV) % period != 0)
    us = []
    for x in (s, p):
        best = np.inf
        for _ in range(4):
            ck.profile_reset()
            ck.profile_enable(True)
            ck.select(spec, x, bud)
            torch.cuda.synchronize()
            ck.profile_enable(False)
            best = min(best, sum(ms for k, (_, ms) in ck.profile_read().items()
                                 if k.startswith("sort")))
        us.append(1e3 * best)
    assert us[1] <= 3 * us[0], us


def _curves(kind, H, n, rng):
    x = np.arange(n, dtype=np.float64)[None]
    scale = rng.uniform(0.1, 10, (H, 1))
    if kind == "noisy_line":
        d = rng.uniform(0.2, 1.8, (H, n))
        c = np.cumsum(d[:, ::-1], 1)[:, ::-1] / n
    elif kind == "noisy_power":
        d = rng.uniform(0.2, 1.8, (H, n)) * (x + 1) ** -rng.uniform(0.3, 1.2, (H, 1))
        c = np.cumsum(d[:, ::-1], 1)[:, ::-1]
    elif kind == "walk":
        c = np.abs(np.cumsum(rng.standard_normal((H, n)), 1))[:, ::-1]
    elif kind == "quantized":  # ties of values, marginals and keys, long plateaus
        c = np.round(np.cumsum(rng.uniform(0, 1, (H, n))[:, ::-1], 1)[:, ::-1] / 16)
        scale = np.ones((H, 1))
    elif kind == "rising":     # the argmin is b_min, the increments all positive
        c = np.cumsum(rng.uniform(0, 1, (H, n)), 1)
    else:                      # "convex": every point on the hull
        c = 1.0 / (1.0 + x / 40.0) + 0 * scale
    return np.ascontiguousarray(c * scale, np.float32)


@pytest.mark.parametrize("kind", ["noisy_line", "noisy_power", "walk", "quantized", "rising",
                                  "convex"])
def test_hull_allocation(kind):
    # Budgets over the hull points against the oracle's full scans: curves of
    # one block and several, chunks of 2048 ranks and their edges, one head to
    # more than a wave each, few and many bisection steps (past the point where
    # the interval has no double inside), every budget size; curves that the
    # hull kernel leaves to the full search among them.
    rng = np.random.default_rng(11)
    for n in (2, 3, 17, 256, 257, 258, 513, 2048, 2049, 2050, 9000):
        for H in ((1, 8) if n != 513 else (3, 17, 40)):
            c = _curves(kind, H, n, rng)
            spec = ck.ProblemSpec(1, H, 1, 64, 1, [n], torch.bfloat16)
            t = torch.from_numpy(c).reshape(1, H, n).to(DEV)
            for n_keep in sorted({2, max(2, n // 10), max(2, n // 2), n}):
                for steps, alpha in ((40, 0.2), (0, 0.2), (9, 0.0), (200, 0.2)):
                    got = ck.allocate_curves(spec, t, [n_keep], steps=steps, alpha=alpha)
                    want, _ = oracle.allocate(c, n_keep, steps=steps, alpha=alpha)
                    assert np.array_equal(got.cpu().numpy(), want), (n, H, n_keep, steps)


@pytest.mark.parametrize("layers", [2, 40, 100])
def test_hull_allocation_beside_the_full_search(layers):
    # One launch with (layer, sequence)s of either kind, for each width of the
    # full search's groups of workgroups.
    rng = np.random.default_rng(layers)
    H, lens = 4, [700, 2333]
    c = np.concatenate([np.stack([_curves("convex" if (li + b) % 3 == 0 else "noisy_power", H, n, rng)
                                  for li in range(layers)]) for b, n in enumerate(lens)], -1)
    spec = ck.ProblemSpec(layers, H, 2, 64, 16, lens, torch.bfloat16)
    n_keep = [71, 240]
    for steps in (0, 5, 40):
        got = ck.allocate_curves(spec, torch.from_numpy(c).to(DEV), n_keep, steps=steps)
        got = got.cpu().numpy().reshape(layers, 2, H)
        for li in range(layers):
            for b, (t0, n) in enumerate(zip((0, lens[0]), lens)):
                want, _ = oracle.allocate(c[li, :, t0:t0 + n], n_keep[b], steps=steps)
                assert np.array_equal(got[li, b], want), (steps, li, b)


@pytest.mark.parametrize("dim,group,tq", [(128, 4, 1), (128, 4, 33), (64, 1, 1), (128, 8, 8),
                                          (128, 8, 40), (64, 8, 32)])
@pytest.mark.parametrize("rows", [[1, 2, 31, 127, 128, 129, 4097, 700], [9000] * 4 + [3] * 5,
                                  [37] * 300, [150000, 10, 4096, 0, 65536],
                                  [128, 128, 256, 0, 0, 1, 127, 0], [0, 5, 300, 0] * 20,
                                  [9001] * 8 + [0] * 60 + [33000] * 60,
                                  [700001, 3, 0, 600000], [5100] * 30, [1100] * 230])
def test_decode_chunks(rows, dim, group, tq):
    # Chunk lengths from 128 to over 4096 keys, chunks that end with a unit and
    # inside one, pieces of one partial and of several, segments of a row to many
    # chunks and empty ones, up to 64 units and more, every piece with a workgroup of
    # its own and not, both combines.  Rows within 1e-4 of fp64 attention, as the
    # decode tests; the same bits under a loose bound on the segments' rows.
    if len(rows) == 300 and dim == 64:
        rows = rows * 30                       # many rows: the row combine
    n = max(max(rows), 16)
    spec = ck.ProblemSpec(1, 1, group, dim, 16, [n] * len(rows))
    gen = torch.Generator(device=DEV).manual_seed(sum(rows) + tq)
    off = torch.tensor([0] + list(np.cumsum(rows)), dtype=torch.int64, device=DEV)
    kp, vp = (torch.randn((sum(rows), dim), generator=gen, device=DEV).bfloat16() for _ in range(2))
    q = torch.randn((1, len(rows) * tq, group, dim), generator=gen, device=DEV).bfloat16()
    out, lse = ck.decode(spec, q, kp, vp, off, tq, with_lse=True, max_rows=max(rows))
    loose = ck.ProblemSpec(1, 1, group, dim, 16, [2 * n + 5000] * len(rows))
    wide = ck.decode(loose, q, kp, vp, off, tq)
    assert torch.equal(wide.nan_to_num(), out.nan_to_num())  # (an empty segment: 0 / 0)
    for u in range(0, len(rows), 1 if len(rows) < 200 else 97):
        a, b = int(off[u]), int(off[u + 1])
        if a == b:
            continue
        x = q[0, u * tq:(u + 1) * tq].double().reshape(tq * group, dim)
        z = (x @ kp[a:b].double().t().contiguous()) / dim ** 0.5
        ref = torch.softmax(z, 1) @ vp[a:b].double()
        got = out[0, u * tq:(u + 1) * tq].double().reshape(tq * group, dim)
        assert ((got - ref).norm(dim=1) <= 1e-4 * ref.norm(dim=1)).all(), u
        err = lse[0, u * tq:(u + 1) * tq].double().reshape(-1) - torch.logsumexp(z, 1)
        assert err.abs().max() <= 1e-4


def test_decode_of_odd_addresses():
    # Cluster summaries and outputs aligned to an element only, in both combines:
    # the same bits as at aligned addresses.
    def shifted(x):
        y = torch.empty(x.numel() + 1, dtype=x.dtype, device=DEV)[1:].reshape(x.shape)
        return y.copy_(x)
    dim, group, m, rows = 128, 4, 5, [300, 41, 2000]
    gen = torch.Generator(device=DEV).manual_seed(3)
    rnd = lambda *s: torch.randn(s, generator=gen, device=DEV)  # noqa: E731
    off = torch.tensor([0] + list(np.cumsum(rows)), dtype=torch.int64, device=DEV)
    kp, vp = rnd(sum(rows), dim).bfloat16(), rnd(sum(rows), dim).bfloat16()
    spec = ck.ProblemSpec(1, 1, group, dim, 16, [2000] * 3, slot=False)
    cl = dict(kbar=(0.1 * rnd(3, m, dim)).bfloat16(), vbar=(0.1 * rnd(3, m, dim)).bfloat16(),
              count=torch.full((3, m), 40, dtype=torch.int32, device=DEV),
              rk=rnd(3, m).abs() * 0.01, rv=rnd(3, m).abs(), vmax_kept=rnd(3).abs() + 15)
    q = rnd(1, 3 * 2, group, dim).bfloat16()
    want = ck.decode_clustered(spec, q, kp, vp, off, 2, cl)
    got = ck.decode_clustered(spec, q, kp, vp, off, 2,
                              dict(cl, kbar=shifted(cl["kbar"]), vbar=shifted(cl["vbar"])))
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    # 8192 rows and more: the combine of several rows to a workgroup
    units, tq = 64, 40
    off = torch.arange(units + 1, device=DEV) * 30
    spec = ck.ProblemSpec(1, 1, group, dim, 16, [30] * units)
    q = rnd(1, units * tq, group, dim).bfloat16()
    bufs = ck.DecodeBuffers(spec, tq, torch.device(DEV))
    want = ck.decode(spec, q, kp[:units * 30], vp[:units * 30], off, tq, bufs=bufs).clone()
    bufs.out = shifted(torch.zeros_like(bufs.out))
    assert bufs.out.data_ptr() % 16 == 4
    assert torch.equal(ck.decode(spec, q, kp[:units * 30], vp[:units * 30], off, tq, bufs=bufs), want)


@pytest.mark.parametrize("tq", [1, 40])
def test_decode_beside_other_units(tq):
    # One sequence's segments alone and inside a ragged batch: other chunks, and so
    # sums grouped otherwise.  Each side applies its weights in 16 bits or better,
    # which bounds the difference at 2 2^-16 of the weighted magnitudes.
    rows, dim, group = [700, 9000, 33, 4100], 128, 4
    more = rows + [20000, 1, 650] * 40
    gen = torch.Generator(device=DEV).manual_seed(7)
    off = torch.tensor([0] + list(np.cumsum(more)), dtype=torch.int64, device=DEV)
    kp, vp = (torch.randn((sum(more), dim), generator=gen, device=DEV).bfloat16() for _ in range(2))
    q = torch.randn((1, len(more) * tq, group, dim), generator=gen, device=DEV).bfloat16()
    got = []
    for r in (rows, more):
        spec = ck.ProblemSpec(1, 1, group, dim, 16, [max(r)] * len(r))
        got.append(ck.decode(spec, q[:, :len(r) * tq].contiguous(), kp[:sum(r)], vp[:sum(r)],
                             off[:len(r) + 1].contiguous(), tq, with_lse=True))
    for u in range(len(rows)):
        a, b = int(off[u]), int(off[u + 1])
        x = q[0, u * tq:(u + 1) * tq].double().reshape(tq * group, dim)
        w = torch.softmax((x @ kp[a:b].double().t().contiguous()) / dim ** 0.5, 1)
        out = [g[0][0, u * tq:(u + 1) * tq].double().reshape(tq * group, dim) for g in got]
        assert ((out[0] - out[1]).abs() <= 2 * 2.0 ** -16 * (w @ vp[a:b].double().abs())).all()
        assert (got[0][1][0, u * tq:(u + 1) * tq] - got[1][1][0, u * tq:(u + 1) * tq]).abs().max() <= 2e-5


@pytest.mark.parametrize("dim,group,window,lens,heads", [
    (64, 1, 1, [1, 63], 2),              # one row, blocks of less than a wave
    (64, 1, 16, [64, 65, 1024, 257], 4),
    (64, 3, 7, [255, 256, 513], 3),      # rows no multiple of the rows per step
    (128, 4, 30, [300, 129], 8),
    (64, 4, 64, [8000, 4097, 9999], 8),  # four-wave blocks, rows not shared out
])
@pytest.mark.parametrize("causal", [True, False])
def test_score_f32_blocks(dim, group, window, lens, heads, causal):
    # fp32 scores, key sums and row log-sum-exps against fp64.  A dot product of
    # dim fp32 terms is off by at most dim 2^-24 times the sum of its terms'
    # magnitudes (under 0.01 here), far above what the sums add.
    spec = ck.ProblemSpec(2, heads, group, dim, window, lens, torch.float32, causal=causal)
    gen = torch.Generator().manual_seed(sum(lens))
    q = torch.randn((2, len(lens) * window, heads * group, dim), generator=gen)
    k = torch.randn((2, sum(lens), heads, dim), generator=gen)
    got, ksum, lse = ck.score(spec, q.to(DEV), k.to(DEV), with_ksum=True, with_lse=True)
    got, ksum, lse = got.cpu().double(), ksum.cpu(), lse.cpu().double()
    given = ck.score(spec, q.to(DEV), k.to(DEV), lse_in=lse.float().to(DEV)).cpu().double()
    t0 = 0
    for b, n in enumerate(lens):
        row = torch.arange(window * group)[:, None] // group
        hide = torch.arange(n)[None] > n - window + row if causal else torch.zeros(1, n).bool()
        for l in range(2):
            for h in range(heads):
                qh = q[l, b * window:(b + 1) * window, h * group:(h + 1) * group].double()
                kh = k[l, t0:t0 + n, h].double()
                z = (qh.reshape(-1, dim) @ kh.t() / dim ** 0.5).masked_fill(hide, -np.inf)
                ref = torch.logsumexp(z, 1)
                x = lse[l, b * window:(b + 1) * window, h * group:(h + 1) * group].reshape(-1)
                assert (x - ref).abs().max() <= 2e-5
                s = (z - ref[:, None]).exp().sum(0)
                assert ((got[l, h, t0:t0 + n] - s).abs() <= 2e-5 * s + 1e-30).all()
                assert ((given[l, h, t0:t0 + n] - s).abs() <= 4e-5 * s + 1e-30).all()
                u = (l * len(lens) + b) * heads + h
                assert ((ksum[u] - s @ kh).abs() <= 4e-5 * (s @ kh.abs())).all()
        t0 += n


@pytest.mark.parametrize("dtype,dim,window", [(torch.bfloat16, 128, 16), (torch.bfloat16, 64, 120),
                                              (torch.float32, 64, 16)])
@pytest.mark.parametrize("lens", [[5000] + [333] * 49 + [1500], [131] * 20 + [9000, 640]])
def test_ragged_key_sums(dtype, dim, window, lens):
    # A long sequence beside short ones, in one launch of up to 48 and in two:
    # the key sums of the scores given out, in fp64.  A block's fp32 sums of at
    # most n terms are off by n 2^-24 of the terms' magnitudes.
    H, G, L = 3, 4 if window > 100 else 2, 2
    spec = ck.ProblemSpec(L, H, G, dim, window, lens, dtype)
    gen = torch.Generator(device=DEV).manual_seed(len(lens))
    q = torch.randn((L, len(lens) * window, H * G, dim), generator=gen, device=DEV).to(dtype)
    k = torch.randn((L, sum(lens), H, dim), generator=gen, device=DEV).to(dtype)
    s, ksum = ck.score(spec, q, k, with_ksum=True)[:2]
    u = torch.arange(L * len(lens) * H).reshape(L, len(lens), H)
    t0 = 0
    for b, n in enumerate(lens):
        sb, kb = s[..., t0:t0 + n].double(), k[:, t0:t0 + n].double()
        for l in range(L):
            for h in range(H):
                ref, mag = sb[l, h] @ kb[l, :, h], sb[l, h] @ kb[l, :, h].abs()
                assert ((ksum[u[l, b, h]] - ref).abs() <= n * 2.0 ** -24 * mag).all(), (l, b, h)
        t0 += n


@pytest.mark.parametrize("name,lens", [("C2", [255, 256, 4097, 20001]), ("C1", [63, 300, 9000])])
def test_gather_splits(name, lens):
    # Kept rows shared out over a unit's splits: none, one, part of a step, a
    # step and a row, and all but one, with the totals given (evicted = totals
    # - kept).  Packed rows are copies.
    # The slot: fp64 sums of n terms in another order, rounded once to fp32;
    # totals minus kept loses the kept share (at most a factor 64 by the rule
    # that sums the evicted rows directly beyond it).
    cfg = synth.config(name, seqlens=lens)
    cache = synth.make_cache(cfg, "cpu")
    spec, H = spec_of(cfg), cfg.kv_heads
    s = _scores((1, H, sum(lens)), 12)
    k, v = cache["k"], cache["v"]
    bud, ksum, vsum, t0 = [], [], [], 0
    for n in lens:
        for h in range(H):
            bud.append([0, 1, min(n, 33), min(n, 129), n // 3, n - 1, n // 50, n // 10][h % 8])
            w = torch.from_numpy(s[0, h, t0:t0 + n]).double()
            ksum.append(w @ k[0, t0:t0 + n, h].double())
            vsum.append(w @ v[0, t0:t0 + n, h].double())
        t0 += n
    st, kd, vd = torch.from_numpy(s).to(DEV), k.to(DEV), v.to(DEV)
    _, off, idx = ck.select(spec, st, torch.tensor(bud, dtype=torch.int32, device=DEV))
    ks, vs, mass = ck.tail_summary(spec, st, kd, vd, off, idx, torch.stack(ksum).to(DEV),
                                   torch.stack(vsum).to(DEV))
    kp, vp, pos, po = ck.compact(spec, kd, vd, off, idx, ks, vs)
    off, po, idx, pos, kp, vp = off.tolist(), po.tolist(), idx.cpu(), pos.cpu(), kp.cpu(), vp.cpu()
    t0 = u = 0
    for b, n in enumerate(lens):
        for h in range(H):
            rows = idx[off[u]:off[u + 1]].long()
            p = po[u]
            assert torch.equal(pos[p:p + len(rows)].long(), rows)
            w = torch.from_numpy(s[0, h, t0:t0 + n]).double()
            tot = w.sum()
            w[rows] = 0.0
            assert abs(mass[u].item() - (w.sum() / tot).item()) <= 1e-12
            for got, packed, x in ((ks, kp, k), (vs, vp, v)):
                x = x[0, t0:t0 + n, h]
                assert torch.equal(packed[p:p + len(rows)], x[rows])
                assert torch.equal(packed[p + len(rows)], got[u].cpu().to(x.dtype))
                z = max(w.sum().item(), 1e-300)  # (nothing evicted: a zero slot)
                ref, scale = w @ x.double() / z, w @ x.double().abs() / z
                assert ((got[u].cpu().double() - ref).abs()
                        <= 2.0 ** -24 * ref.abs() + 64 * n * 2.0 ** -52 * scale + 1e-300).all(), u
            u += 1
        t0 += n


def test_kept_bitmap_of_unordered_positions():
    # Kept positions of a caller's own, not ascending, repeated or out of range:
    # the evicted mass is that of the positions in none of them.
    n, H = 700, 4
    spec = ck.ProblemSpec(1, H, 1, 64, 16, [n], torch.float32)
    gen = torch.Generator().manual_seed(2)
    idx = torch.stack([torch.randperm(n, generator=gen)[:300], torch.arange(300).flip(0),
                       torch.arange(300) // 3 * 5 % n,
                       torch.arange(300) % 2 * 64 + torch.arange(300) % 7]).int()
    idx[3, 5] = -1
    idx[3, 6] = n
    s = torch.rand((1, H, n), generator=gen) + 0.5
    k = torch.randn((1, n, H, 64), generator=gen)
    off = torch.arange(H + 1, dtype=torch.int64) * 300
    _, _, mass = ck.tail_summary(spec, s.to(DEV), k.to(DEV), k.to(DEV), off.to(DEV),
                                 idx.reshape(-1).to(DEV))
    for h in range(H):
        w = s[0, h].double()
        tot = w.sum()
        ok = idx[h][(idx[h] >= 0) & (idx[h] < n)].long()
        w[ok] = 0.0
        assert abs(mass[h].item() - (w.sum() / tot).item()) <= 1e-12


@pytest.mark.parametrize("lens,heads,layers", [
    ([8192, 8191, 1], 4, 1), ([8193, 40960, 24577], 4, 1),  # parts of one tile, and their edges
    ([65537, 9000], 8, 6),                                  # parts of several
    ([16400], 8, 32),                                       # a unit per compute unit: not split
])
@pytest.mark.parametrize("keep_window", [False, True])
def test_select_parts(lens, heads, layers, keep_window):
    # Kept positions and masks of budgets from none to all against the order.
    rng = np.random.default_rng(len(lens))
    w = 1 if min(lens) < 16 else 16
    spec = ck.ProblemSpec(layers, heads, 1, 64, w, lens, torch.float32, keep_window=keep_window)
    s = np.round(_scores((layers, heads, sum(lens)), 9) * 64) / 64  # ties across parts
    bud = np.array([[[rng.integers(0, n + 1) for _ in range(heads)] for n in lens]
                    for _ in range(layers)], np.int32)
    bud[0, :, 0], bud[0, :, 1] = 0, lens
    got, off, idx, mask = ck.select(spec, torch.from_numpy(s).to(DEV),
                                    torch.from_numpy(bud.reshape(-1)).to(DEV), with_mask=True)
    off, idx, mask = off.tolist(), idx.cpu().numpy(), mask.cpu().numpy()
    u, step = 0, 1 if layers < 10 else 7
    for l in range(layers):
        t0 = 0
        for b, n in enumerate(lens):
            for h in range(heads):
                assert off[u + 1] - off[u] == bud[l, b, h]
                if u % step == 0:
                    perm = oracle.order(s[l, h, t0:t0 + n], keep_window=w if keep_window else 0)
                    kept = np.sort(perm[:bud[l, b, h]])
                    assert np.array_equal(idx[off[u]:off[u + 1]], kept), (l, b, h)
                    ref = np.zeros(n, np.uint8)
                    ref[kept] = 1
                    assert np.array_equal(mask[l, h, t0:t0 + n], ref)
                u += 1
            t0 += n


@pytest.mark.parametrize("layers,heads,batch", [(1, 1, 1), (16, 8, 8), (5, 41, 5), (2, 8, 70)])
def test_offsets_of_many_units(layers, heads, batch):
    # Offsets summed by the selection (up to 1024 units, several launches of 48
    # sequences) and by a launch of their own; no key kept at the ends.
    lens = [17 + 3 * (b % 5) for b in range(batch)]
    spec = ck.ProblemSpec(layers, heads, 1, 64, 16, lens, torch.float32)
    rng = np.random.default_rng(layers)
    bud = np.concatenate([rng.integers(0, 17, heads) for _ in range(layers * batch)]).astype(np.int32)
    bud[0] = bud[-1] = 0
    s = torch.from_numpy(_scores((layers, heads, sum(lens)), 4)).to(DEV)
    _, off, idx = ck.select(spec, s, torch.from_numpy(bud).to(DEV))
    assert np.array_equal(off.cpu().numpy(), np.concatenate([[0], np.cumsum(bud)]))
    off, idx, s = off.tolist(), idx.cpu().numpy(), s.cpu().numpy()
    starts = np.concatenate([[0], np.cumsum(lens)])
    for u in range(len(bud)):
        l, b, h = u // (batch * heads), u // heads % batch, u % heads
        sh = s[l, h, starts[b]:starts[b + 1]]
        assert np.array_equal(idx[off[u]:off[u + 1]], np.sort(oracle.order(sh)[:bud[u]]))
