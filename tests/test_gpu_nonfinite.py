"""Infinite and NaN values in the cache and among the new pairs: a pair of weight p > 0 gives p * inf = inf in its channel, whatever form the weights take in the
kernel; every other channel is what it is without it."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util
    import paper_2602_03203_amd as fk
    fk.lib()
    return gpu_util


DT = {"bf16": torch.bfloat16, "f32": torch.float32}
INF, NAN = float("inf"), float("nan")
B, H, G, T = 2, 2, 4, 12


def run(fk, form, desc, args, ml, scale):
    """Outputs [T][B][heads][D] of T steps, and the feature state."""
    q, K, V, pos, ln, k, v, pn = (a.clone() for a in args)
    out = torch.zeros_like(q)
    feat = fk.new_feat(desc) if "feat" in form else None
    ws = fk.new_feat_workspace(desc) if "feat" in form else fk.new_attn_workspace(desc)
    if form == "window":
        fk.fk_decode_window(desc, q, K, V, pos, ln, k, v, pn, T, ml, scale, out, ws)
    elif form == "window_feat":
        fk.fk_decode_window_feat(desc, q, K, V, pos, ln, k, v, pn, T, ml, scale, feat, 0, 32, out, ws)
    for t in range(0 if "window" in form else T):
        a = (desc, q[t], K, V, pos, ln, k[t], v[t], pn[t], ml + t, scale)
        if form == "step":
            fk.fk_decode_step(*a, out[t], ws)
        elif form == "static":
            fk.fk_decode_step_static(*a, out[t])
        elif form == "step_feat":
            fk.fk_decode_step_feat(*a, feat, t, 32, out[t], ws)
        else:   # append, attend
            fk.fk_append(desc, K, V, pos, ln, k[t], v[t], pn[t])
            fk.fk_decode_attn(desc, q[t], K, V, ln, ml + t, scale, out[t], ws)
    torch.cuda.synchronize()
    return out.float(), feat


# rows of one split and of several; the workgroup that holds the infinity has keys before and behind it
@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("n", [160, 1500])
@pytest.mark.parametrize("form", ["step", "static", "attn", "step_feat", "window", "window_feat"])
def test_infinite_cached_values(gpu, dtype, D, n, form):
    import paper_2602_03203_amd as fk
    print(f"infinite values {dtype} D={D} n={n} {form}", flush=True)
    cap = n + 20
    desc = fk.CacheDesc(B, H * G, H, D, cap, dtype)
    gen = torch.Generator(device="cuda").manual_seed(n + D)
    mk = lambda *s: torch.randn(s, generator=gen, device="cuda").to(DT[dtype])   # noqa: E731
    q, K, V, k, v = mk(T, B, H * G, D), mk(B, H, cap, D), mk(B, H, cap, D), mk(T, B, H, D), mk(T, B, H, D)
    K[0, 1, 45] = 4.0 * q[3, 0, H * G // 2]   # the largest weight of a row (1 before the division): nothing left for a remainder
    pos = torch.arange(cap, dtype=torch.int32, device="cuda").expand(B, H, cap).contiguous()
    ln, pn = torch.full((B, H), n, dtype=torch.int32, device="cuda"), torch.zeros((T, B), dtype=torch.int32, device="cuda")
    bad = [(0, 1, 45, 17, INF), (0, 1, 46, 18, -INF), (0, 1, 47, 19, NAN), (1, 0, 5, 3, INF), (1, 0, 101, 4, -INF), (1, 0, 70, 3, INF)]
    clean = V.clone()
    for b, h, slot, c, x in bad:
        V[b, h, slot, c] = x
        clean[b, h, slot, c] = 0.0
    o = run(fk, form, desc, (q, K, V, pos, ln, k, v, pn), n + 1, 0.1)[0]
    r = run(fk, form, desc, (q, K, clean, pos, ln, k, v, pn), n + 1, 0.1)[0]
    for b, h, _, c, x in bad:
        got = o[:, b, h * G:(h + 1) * G, c]
        assert bool(torch.isnan(got).all() if x != x else (got == x).all()), f"row ({b},{h}) channel {c}: {got.flatten()[:4]} for {x}"
    for b, h, _, c, _ in bad:
        o[:, b, h * G:(h + 1) * G, c] = r[:, b, h * G:(h + 1) * G, c]
    assert torch.equal(o, r)


# the pair of step 5 is the row's last one then: at a tile's end (n = 90: slot 95) and inside a tile, where the lanes past the end hold copies of it
@pytest.mark.parametrize("dtype,D", [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("n", [90, 70, 1500])
@pytest.mark.parametrize("form", ["step", "static", "attn", "step_feat", "window", "window_feat"])
def test_infinite_new_values(gpu, dtype, D, n, form):
    import paper_2602_03203_amd as fk
    print(f"infinite new values {dtype} D={D} n={n} {form}", flush=True)
    cap = n + 20
    desc = fk.CacheDesc(B, H * G, H, D, cap, dtype)
    gen = torch.Generator(device="cuda").manual_seed(n + D)
    mk = lambda *s: torch.randn(s, generator=gen, device="cuda").to(DT[dtype])   # noqa: E731
    q, K, V, k, v = mk(T, B, H * G, D), mk(B, H, cap, D), mk(B, H, cap, D), mk(T, B, H, D), mk(T, B, H, D)
    pos = torch.arange(cap, dtype=torch.int32, device="cuda").expand(B, H, cap).contiguous()
    ln, pn = torch.tensor([[n, n - 3], [n, n]], dtype=torch.int32, device="cuda"), torch.zeros((T, B), dtype=torch.int32, device="cuda")
    bad = [(5, 0, 0, 17, INF), (5, 0, 0, 18, -INF), (6, 0, 0, 19, NAN), (5, 0, 1, 3, INF), (7, 1, 0, 3, -INF), (11, 1, 0, 40, NAN)]
    clean = v.clone()
    for t, b, h, c, x in bad:
        v[t, b, h, c] = x
        clean[t, b, h, c] = 0.0
    o, f = run(fk, form, desc, (q, K, V, pos, ln, k, v, pn), n + 1, 0.1)
    r, fr = run(fk, form, desc, (q, K, V, pos, ln, k, clean, pn), n + 1, 0.1)
    for t, b, h, c, x in bad:
        got = o[t:, b, h * G:(h + 1) * G, c]
        assert bool(torch.isnan(got).all() if x != x else (got == x).all()), f"row ({b},{h}) channel {c} from step {t}: {got[:, 0]} for {x}"
    for t, b, h, c, _ in bad:
        o[t:, b, h * G:(h + 1) * G, c] = r[t:, b, h * G:(h + 1) * G, c]
    assert torch.equal(o, r)
    assert f is None or torch.equal(f, fr)
