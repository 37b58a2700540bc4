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


# the bound of a split selection: right, too high for every pair but the sampled ones (the merge starts over), with all of the best in one chunk,
# among ties, and useless; rows too short for a sample; a length hint below the length (the last chunk is longer than the others)
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
