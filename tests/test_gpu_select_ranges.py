"""Selection where the histogram over the keys' range can go wrong: value distributions that crowd one bin, both signs, infinities and NaN,
ranges of a few bits, and row lengths around the workgroup's, against the oracle."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from util import random_cache

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util
    import paper_2602_03203_amd as fk
    fk.lib()
    return gpu_util


def values(kind, n, seed):
    z = si.normal(seed, si.T_SCORE, 0, np.arange(n)).astype(np.float32)
    s = z.copy()
    if kind == "positive":
        s = np.exp(z)
    elif kind == "negative":
        s = -np.exp(3 * z)
    elif kind == "outlier":           # all but two keys share one bin
        s[n // 3], s[n // 2] = 1e30, -1e30
    elif kind == "heavy tails":       # a range far wider than what most keys span
        s = (z / (np.abs(np.roll(z, 1)) + np.float32(1e-4))).astype(np.float32)
    elif kind == "one end":           # one wavefront's keys far from the others'
        s[: n // 16] += np.float32(1e6)
    elif kind == "huge":              # the difference of the extremes overflows
        s[n // 3], s[n // 2] = 3.4e38, -3.4e38
    elif kind == "infinite":
        s[::7], s[3::11] = np.inf, -np.inf
    elif kind == "nan":
        s[::5] = np.nan
    elif kind == "denormal":          # both signs, a range below the smallest normal number
        s = (z * 1e-40).astype(np.float32)
    elif kind == "bits":              # neighbours of 1.0, many ties
        s = (np.float32(1.0).view(np.uint32) + (si.hash_u64(seed, 1, 0, np.arange(n)) % np.uint64(37)).astype(np.uint32)).view(np.float32)
    elif kind == "zeros":             # -0 and +0 are equal
        s = np.where(z > 0.5, z, np.where(z > 0, np.float32(0.0), np.float32(-0.0))).astype(np.float32)
    elif kind == "two":
        s = np.where(z > 0, np.float32(2.5), np.float32(-1.0)).astype(np.float32)
    elif kind == "equal":
        s[:] = -3.0
    return s


KINDS = ["normal", "positive", "negative", "outlier", "heavy tails", "one end", "huge", "infinite", "nan", "denormal", "bits", "zeros", "two", "equal"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n,budget,recent", [(2176, 2048, 128), (1025, 64, 0), (130, 100, 16), (273, 200, 16), (272, 200, 16), (5000, 1, 0), (9000, 2500, 100)])
def test_selection_over_value_ranges(gpu, ora, kind, n, budget, recent):
    import paper_2602_03203_amd as fk
    print(f"select {kind} n={n} budget={budget} recent={recent}", flush=True)
    c = random_cache(ora, 5, "bf16", 1, 2, n, 64, lens=[n])
    desc = fk.CacheDesc(1, 2, 2, 64, n, "bf16")
    sc = np.stack([values(kind, n, 40 + h) for h in range(2)])[None]
    noise = si.gen_gumbel(77, (1, 2, n))
    pos, ln = gpu.to_dev(c.pos), torch.full((1, 2), n, dtype=torch.int32, device="cuda")
    keep = torch.full((1, 2, budget), -1, dtype=torch.int32, device="cuda")
    fk.fk_select_keep(desc, gpu.to_dev(sc), pos, ln, n, budget, recent, keep)
    gpu.assert_keep_equal(keep.cpu().numpy(), ora.select_keep(sc, c.pos, c.len, budget, recent, "sort"), c.len, budget, kind)
    if kind != "nan":   # score - noise is a number or an infinity
        fk.fk_select_keep_sampled(desc, gpu.to_dev(sc), gpu.to_dev(noise), pos, ln, n, budget, recent, 2 * (n - budget), keep)
        ref = ora.select_keep_sampled(sc, noise, c.pos, c.len, budget, recent, 2 * (n - budget))
        gpu.assert_keep_equal(keep.cpu().numpy(), ref, c.len, budget, kind + " sampled")


@pytest.mark.parametrize("n", [5000, 8192 + 16, 20000])
@pytest.mark.parametrize("m,step", [(40, 1), (64, 3), (150, 0), (150, 2), (230, 1), (256, 1), (300, 1)])
def test_cut_in_a_full_bin(gpu, ora, n, m, step):
    """m keys a few bits apart (0: equal) around the cut, beside some of the others in its bin: below, at and beyond what is ranked as a list."""
    import paper_2602_03203_amd as fk
    print(f"select full bin n={n} m={m} step={step}", flush=True)
    recent = 16
    sc = np.stack([values("normal", n, 80 + h) for h in range(2)])
    for h in range(2):
        where = (np.arange(m) * 19 + 5 * h + 1) % (n - recent)
        sc[h, where] = (np.float32(0.25).view(np.uint32) + np.uint32(step) * (np.arange(m, dtype=np.uint32) * 7 % m)).view(np.float32)
    budget = int((sc[0, : n - recent] > 0.25 + 1e-4).sum()) + m // 2 + recent
    c = random_cache(ora, 7, "bf16", 1, 2, n, 64, lens=[n])
    desc = fk.CacheDesc(1, 2, 2, 64, n, "bf16")
    pos, ln = gpu.to_dev(c.pos), torch.full((1, 2), n, dtype=torch.int32, device="cuda")
    keep = torch.full((1, 2, budget), -1, dtype=torch.int32, device="cuda")
    fk.fk_select_keep(desc, gpu.to_dev(sc[None]), pos, ln, n, budget, recent, keep)
    gpu.assert_keep_equal(keep.cpu().numpy(), ora.select_keep(sc[None], c.pos, c.len, budget, recent, "sort"), c.len, budget, "full bin")


@pytest.mark.parametrize("kind", ["normal", "positive", "outlier", "bits", "infinite"])
def test_split_selection_over_value_ranges(gpu, ora, kind):
    import paper_2602_03203_amd as fk
    n, budget, recent = 20011, 1500, 33
    c = random_cache(ora, 6, "bf16", 1, 2, n, 64, lens=[n])
    desc = fk.CacheDesc(1, 2, 2, 64, n, "bf16")
    sc = np.stack([values(kind, n, 60 + h) for h in range(2)])[None]
    need = fk.fk_select_keep_workspace(desc, n, budget, recent)
    assert need > 0
    keep = torch.full((1, 2, budget), -1, dtype=torch.int32, device="cuda")
    fk.fk_select_keep_ws(desc, gpu.to_dev(sc), None, torch.full((1, 2), n, dtype=torch.int32, device="cuda"), n, budget, recent, keep,
                         torch.empty(need, dtype=torch.uint8, device="cuda"))
    gpu.assert_keep_equal(keep.cpu().numpy(), ora.select_keep(sc, c.pos, c.len, budget, recent, "sort"), c.len, budget, kind)


def sampled_slots(n_cand):
    """The slots whose scores a split selection looks at for its bound: one of each of 2048 stretches, placed by a hash (fp32, as on the device)."""
    i = np.arange(2048, dtype=np.uint32)
    frac = ((i * np.uint32(2654435761)) >> np.uint32(8)).astype(np.float32) * np.float32(1 / 16777216)
    return np.minimum(((i.astype(np.float32) + frac) * (np.float32(n_cand) / np.float32(2048))).astype(np.int64), n_cand - 1)


def split_plan(rows, hint, budget, recent):
    """(chunks of a row, pairs of a chunk but the last) as the library cuts rows for fk_select_keep_ws."""
    nchunk = min(256 // rows, 18 * 1024 // (budget - recent), 16)
    return nchunk, ((hint - recent + nchunk - 1) // nchunk + 3) // 4 * 4


def looks_for_bound(n, chunk_len, budget, recent):
    """Whether the chunks of a row of n pairs look for a bound, and how many of the 2048 sampled scores reach it."""
    mean = 2048 * (budget - recent) / (n - recent)
    reach = int(mean + 6 * np.sqrt(mean)) + 8
    return n - recent >= 8 * 2048 and 4 * reach <= 2048 and chunk_len >= 2048, reach


# the bound of a split selection: right, too high for every pair but the sampled ones (the merge starts over), with all of the best in one chunk,
# among ties, and useless; rows too short for a sample; the last shape has chunks too short for one
@pytest.mark.parametrize("kind", ["normal", "sampled", "one chunk", "ramp", "two", "equal", "nan", "infinite"])
@pytest.mark.parametrize("n,lens,hint,budget,recent", [(70001, [70001, 20000, 16500, 900], 70001, 700, 16), (131072, [131072, 131071, 60000, 16384 + 128], 131072, 2048, 128),
                                                       (40000, [40000, 39000, 30000, 20000], 20000, 300, 0)])
def test_split_selection_by_a_sampled_bound(gpu, ora, kind, n, lens, hint, budget, recent):
    import paper_2602_03203_amd as fk
    sc = np.stack([values(kind, n, 80 + b) for b in range(4)])[:, None]
    for b in range(4):
        if kind == "sampled" and lens[b] > budget:
            sc[b, 0, sampled_slots(lens[b] - recent)] += 100.0
        elif kind == "one chunk":
            sc[b, 0, lens[b] // 3: lens[b] // 3 + budget] += 100.0
        elif kind == "ramp":
            sc[b, 0] += np.arange(n, dtype=np.float32) / 1000
    pos, ln = np.broadcast_to(np.arange(n, dtype=np.int32), (4, 1, n)), np.array(lens, np.int32)
    desc = fk.CacheDesc(4, 1, 1, 64, n, "bf16")
    need = fk.fk_select_keep_workspace(desc, hint, budget, recent)
    assert need > 0
    print(f"sampled bound {kind} {lens} hint {hint} budget {budget}", flush=True)
    keep = torch.full((4, 1, budget), -1, dtype=torch.int32, device="cuda")
    fk.fk_select_keep_ws(desc, gpu.to_dev(sc), None, torch.from_numpy(ln[:, None].copy()).cuda(), hint, budget, recent, keep, torch.empty(need, dtype=torch.uint8, device="cuda"))
    gpu.assert_keep_equal(keep.cpu().numpy(), ora.select_keep(sc, np.ascontiguousarray(pos), ln, budget, recent, "sort"), ln, budget, kind)


# The bound in chunks that a workgroup cannot hold in registers (more than 16384 pairs), in LDS and in global memory, because there are
# few chunks or because the last one runs on to the end of a row longer than the hint; rows in multiples of eight, whose chunks are dealt
# to the XCDs in another order; "over" says of the first row's last chunk whether normal scores leave it with more pairs over the bound than
# it may pass on.  "coarse": the cut goes through equal scores, of which a chunk has more than it may pass on, but not above them.
@pytest.mark.parametrize("kind", ["normal", "sampled", "one chunk", "ramp", "two", "equal", "coarse", "infinite"])
@pytest.mark.parametrize("batch,hkv,n,lens,hint,budget,recent,last,over", [
    (8, 8, 131072, None, 131072, 1930, 10, "lds", False),               # 4 chunks of 32768
    (8, 1, 131072, None, 131072, 4432, 32, "lds", False),               # 4 chunks of 32768, kept lists that fill the merge
    (1, 2, 131072, [131072], 131072, 9100, 100, "global", False),       # 2 chunks of 65536
    (2, 1, 90000, [90000, 61000], 60000, 3000, 100, "global", False),   # a last chunk of 40000
    (2, 1, 90000, [90000, 60000], 40000, 3000, 100, "global", True),    # ... of 56000
    (1, 4, 90000, [90000], 40000, 300, 0, "global", True),              # 15 chunks of 2500 and one of 52500
    (24, 1, 40000, None, 40000, 333, 33, "registers", False),           # 24 rows, 10 chunks
    (2, 4, 33000, [33000, 25001], 33000, 900, 7, "registers", False),   # 8 rows, 16 chunks
])
def test_split_selection_bound_in_long_chunks(gpu, ora, kind, batch, hkv, n, lens, hint, budget, recent, last, over):
    import paper_2602_03203_amd as fk
    rows = batch * hkv
    lens = lens or [n - 1000 * b for b in range(batch)]
    nchunk, chunk_len = split_plan(rows, hint, budget, recent)
    tail = lens[0] - recent - (nchunk - 1) * chunk_len
    found, reach = looks_for_bound(lens[0], chunk_len, budget, recent)
    assert found and last == ("registers" if tail <= 16384 else "lds" if tail <= min(chunk_len, 36 * 1024) else "global")
    expected = reach / 2048 * tail   # pairs of the tail that reach the bound
    assert expected > 1.1 * (budget - recent) if over else expected < 0.9 * (budget - recent)
    base = np.stack([values("two" if kind == "two" else "equal" if kind == "equal" else "infinite" if kind == "infinite" else "normal", n, 300 + r) for r in range(min(rows, 8))])
    sc = np.stack([np.roll(base[r % 8], 977 * r) for r in range(rows)]).reshape(batch, hkv, n)   # every row its own
    for b in range(batch):
        if kind == "sampled":
            sc[b][:, sampled_slots(lens[b] - recent)] += 100.0
        elif kind == "one chunk":
            sc[b][:, lens[b] // 3: lens[b] // 3 + budget] += 100.0
        elif kind == "ramp":
            sc[b] += np.arange(n, dtype=np.float32) / 1000
        elif kind == "coarse":
            sc[b] = np.round(sc[b])
    desc = fk.CacheDesc(batch, hkv, hkv, 64, n, "bf16")
    need = fk.fk_select_keep_workspace(desc, hint, budget, recent)
    assert need >= rows * nchunk * (budget - recent + 1) * 4
    print(f"bound in long chunks {kind} {batch}x{hkv} {lens} hint {hint} budget {budget}", flush=True)
    pos, ln = np.broadcast_to(np.arange(n, dtype=np.int32), (batch, hkv, n)), np.array(lens, np.int32)
    keep = torch.full((batch, hkv, budget), -1, dtype=torch.int32, device="cuda")
    work = torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda")
    d_len = torch.from_numpy(np.repeat(ln[:, None], hkv, axis=1)).cuda()
    fk.fk_select_keep_ws(desc, gpu.to_dev(sc), None, d_len, hint, budget, recent, keep, work)
    gpu.assert_keep_equal(keep.cpu().numpy(), ora.select_keep(sc, np.ascontiguousarray(pos), ln, budget, recent, "sort"), ln, budget, kind)


@pytest.mark.parametrize("budget", [1, 255, 256, 257, 511, 512, 513, 1024, 1025, 1537, 2200])
@pytest.mark.parametrize("features", [0, 4, 8])
def test_compact_over_the_edges_of_its_tiles(gpu, budget, features):
    """Budgets around one, two, three and four tiles of 256 and 512 slots: rows that move by one slot, by a tile and one, at random, only behind
    a tile, and not at all; every slot of cache and positions, the carried feature sums with them, exactly."""
    import paper_2602_03203_amd as fk
    print(f"compact budget {budget} features {features}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(budget)
    n, g = budget + 600, max(features, 1)
    desc = fk.CacheDesc(5, g, 1, 64, n, "bf16")
    K, V = (torch.randint(-30000, 30000, (5, 1, n, 64), generator=gen, device="cuda", dtype=torch.int16).view(torch.bfloat16) for _ in range(2))
    pos = torch.arange(5 * n, dtype=torch.int32, device="cuda").reshape(5, 1, n)
    j = torch.arange(budget, device="cuda")
    rand = torch.randperm(n, generator=gen, device="cuda")[:budget].sort().values
    keep = torch.stack([j + 1, j + min(513, 600), rand, torch.where(j >= min(513, budget - 1), j + 300, j), j]).int().reshape(5, 1, budget).contiguous()
    ln = torch.full((5, 1), n, dtype=torch.int32, device="cuda")
    want = [x.clone() for x in (K, V, pos)]
    for x, y in zip(want, (K, V, pos)):
        for r in range(5):
            x[r, 0, :budget] = y[r, 0, keep[r, 0].long()]
    if features:
        feat = torch.rand((5, 1, 6, n, fk.feat_heads(desc)), generator=gen, device="cuda")
        f0 = feat.clone()
        fk.fk_compact_feat(desc, K, V, pos, feat, ln, keep, budget)
        for r in range(5):
            i = keep[r, 0].long()
            assert torch.equal(feat[r, 0, 4, :budget], f0[r, 0, 4, i] + f0[r, 0, 3, i]) and not feat[r, 0, :4].any()
    else:
        fk.fk_compact(desc, K, V, pos, ln, keep, budget)
    assert ln.eq(budget).all()
    for x, y in zip(want, (K, V, pos)):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))


# rows of head_dim 64 (two workgroups each): up to 192 workgroups look for the first slot that moves beyond the first two tiles (1024 slots), in
# passes of 4096 slots from there; up to 256 and beyond do not
@pytest.mark.parametrize("rows,budget", [(12, 1025), (12, 1537), (12, 5121), (12, 9300), (80, 1700), (96, 1500), (97, 1500), (128, 1500), (129, 1500)])
@pytest.mark.parametrize("holes", [False, True])
def test_compact_of_rows_that_move_late(gpu, rows, budget, holes):
    """Rows that stay up to a slot at the edges of tiles and passes, and rows that stay for good; with holes, every second slot that stays has an index
    outside the cache instead of its own."""
    import paper_2602_03203_amd as fk
    print(f"compact late rows {rows} budget {budget} holes {holes}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(budget)
    n = budget + 40
    desc = fk.CacheDesc(rows, 1, 1, 64, n, "bf16")
    K, V = (torch.randint(-30000, 30000, (rows, 1, n, 64), generator=gen, device="cuda", dtype=torch.int16).view(torch.bfloat16) for _ in range(2))
    pos = torch.arange(rows * n, dtype=torch.int32, device="cuda").reshape(rows, 1, n)
    edges = [0, 511, 512, 1023, 1024, 1025, 1535, 1536, 5119, 5120, 9216, budget - 1, budget]
    first = torch.tensor([min(edges[r % len(edges)], budget) for r in range(rows)], device="cuda")
    j = torch.arange(budget, device="cuda")
    stays = j[None, :] < first[:, None]
    keep = torch.where(stays, j, j + 1 + torch.arange(rows, device="cuda")[:, None] % 40)
    src = keep.clone()
    if holes:
        keep = torch.where(stays & (j % 2 == 1), torch.where(j % 4 == 1, -1, n + j), keep)
    keep = keep.int().reshape(rows, 1, budget).contiguous()
    ln = torch.full((rows, 1), n, dtype=torch.int32, device="cuda")
    want = [x.clone() for x in (K, V, pos)]
    for x, y in zip(want, (K, V, pos)):
        i = src.reshape(src.shape + (1,) * (y.dim() - 3)).expand((rows, budget) + y.shape[3:])
        x[:, 0, :budget] = y[:, 0].gather(1, i)
    fk.fk_compact(desc, K, V, pos, ln, keep, budget)
    assert ln.eq(budget).all()
    for x, y in zip(want, (K, V, pos)):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))
