"""The softmax over its whole range: logits of any size, negative and zero scales, hidden pairs; steps, windows and feature planes."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_03203_amd as fk
    fk.lib()
    return fk


def steps_and_window(fk, desc, q, K, V, ln, k, v, scale, feat=False):
    """Outputs (and planes) of the single steps; those of fk_decode_window have to be the same bits."""
    T, res = q.shape[0], []
    pos = torch.zeros(K.shape[:3], dtype=torch.int32, device="cuda")
    pn = torch.zeros((T, desc.batch), dtype=torch.int32, device="cuda")
    ml = int(ln.max()) + 1
    for window in (False, True):
        Kc, Vc, pc, lc, out = K.clone(), V.clone(), pos.clone(), ln.clone(), torch.zeros_like(q)
        if feat:
            F, ws = fk.new_feat(desc), fk.new_feat_workspace(desc)
            if window:
                fk.fk_decode_window_feat(desc, q, Kc, Vc, pc, lc, k, v, pn, T, ml, scale, F, 0, T, out, ws)
            for t in range(0 if window else T):
                fk.fk_decode_step_feat(desc, q[t], Kc, Vc, pc, lc, k[t], v[t], pn[t], ml + t, scale, F, t, T, out[t], ws)
            res.append((out, F))
        else:
            ws = fk.new_attn_workspace(desc)
            if window:
                fk.fk_decode_window(desc, q, Kc, Vc, pc, lc, k, v, pn, T, ml, scale, out, ws)
            for t in range(0 if window else T):
                fk.fk_decode_step(desc, q[t], Kc, Vc, pc, lc, k[t], v[t], pn[t], ml + t, scale, out[t], ws)
            res.append((out,))
    for a, b in zip(*res):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), "window and steps differ"
    return res[0]


# The logits are scale * D * size^2, so up to 1.4e25, plus and minus: 2^23 and 2^24 are where a product and its rounding are a unit apart, 2^32 where
# they are more than an exponential's range.  700 pairs of few rows are split.
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rows,g,n", [(128, 4, 45), (4, 4, 700), (128, 1, 300), (4, 7, 45)])
@pytest.mark.parametrize("size", [96.0, 1536.0, 14336.0, 24576.0, 28672.0, 2.0 ** 40])
@pytest.mark.parametrize("sign", [1, -1])
def test_equal_and_dominating_pairs_at_any_size(gpu, D, rows, g, n, size, sign):
    """Pairs of the largest logit share the weight equally, the others, one or two sizes below, have none.  All products and sums of a logit are
    exact in fp32 (a few significant bits, a power of two of equal terms), and so are equal weights and their sum: what is left is the division
    and the rounding to bf16."""
    fk = gpu
    T, cap = 6, n + 6
    print(f"softmax range D={D} rows={rows} g={g} n={n} size={size} sign={sign}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n + g)
    desc = fk.CacheDesc(rows, g, 1, D, cap, "bf16")
    top = torch.zeros((rows, cap), dtype=torch.bool, device="cuda")
    ln = torch.full((rows, 1), n, dtype=torch.int32, device="cuda")
    ln[0] = 0                                                    # only the new pairs, all equal (below)
    top[0] = True
    for r in range(1, rows):                                     # one, two, three equal ones in other places of other tiles
        top[r, [(7 * r) % n, n - 1, n // 2][:1 + r % 3]] = True
    key = torch.where(top, size, torch.where(torch.arange(cap, device="cuda") % 2 == 0, -size, 0.0))
    K = (sign * key[:, None, :, None]).expand(rows, 1, cap, D).to(torch.bfloat16).contiguous()
    V = torch.randn((rows, 1, cap, D), generator=gen, device="cuda").to(torch.bfloat16)
    q = torch.full((T, rows, g, D), size, device="cuda", dtype=torch.bfloat16)
    k = torch.full((T, rows, 1, D), -sign * size, device="cuda", dtype=torch.bfloat16)
    k[:, 0] = sign * size
    v = torch.randn((T, rows, 1, D), generator=gen, device="cuda").to(torch.bfloat16)
    out, = steps_and_window(fk, desc, q, K, V, ln, k, v, sign * D ** -0.5)
    top[0], w = False, None
    for t in range(T):
        V[0, 0, t], top[0, t] = v[t, 0, 0], True
        w = top.double() / top.sum(1, keepdim=True)
        ref = (w[:, None, :] @ V[:, 0].double()).expand(rows, g, D)
        off = (out[t].double() - ref).abs() - 2.0 ** -8 * ref.abs() - 1e-6
        assert bool((off <= 0).all()), f"step {t}: {out[t].isnan().sum().item()} NaN, worst {off.max().item():.3g}"


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("rows,n", [(128, 45), (4, 700)])
@pytest.mark.parametrize("size", [1.0, 1e18])
def test_scale_zero_is_the_mean(gpu, D, rows, n, size):
    """Logits of up to 1.3e38 times 0 are 0: every pair has the same weight, hidden ones have none."""
    fk = gpu
    T, g = 6, 4
    gen = torch.Generator(device="cuda").manual_seed(n)
    desc = fk.CacheDesc(rows, g, 1, D, n + T, "bf16")
    sgn = lambda *s: torch.randint(0, 2, s, generator=gen, device="cuda").mul(2).sub(1).float()   # noqa: E731
    K = (sgn(rows, 1, n + T, 1) * size).expand(rows, 1, n + T, D).to(torch.bfloat16).contiguous()
    V = torch.randn((rows, 1, n + T, D), generator=gen, device="cuda").to(torch.bfloat16)
    q = torch.full((T, rows, g, D), size, device="cuda", dtype=torch.bfloat16)
    k = (sgn(T, rows, 1, 1) * size).expand(T, rows, 1, D).to(torch.bfloat16).contiguous()
    v = torch.randn((T, rows, 1, D), generator=gen, device="cuda").to(torch.bfloat16)
    ln = torch.full((rows, 1), n, dtype=torch.int32, device="cuda")
    out, = steps_and_window(fk, desc, q, K, V, ln, k, v, 0.0)
    for t in range(T):
        V[:, :, n + t] = v[t]
        ref = V[:, :, :n + t + 1].double().mean(2).expand(rows, g, D)
        assert bool(((out[t].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5).all())   # (1e-5: n fp32 additions of values up to 5)


# In units of 2^-24: an exponential twice (2 each), at most 24 corrections by another (3 each), 1 / l, two products and the sum over the pairs in fp32
FEAT_SUM = 128 * 2.0 ** -24


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("g", [1, 4, 8])
@pytest.mark.parametrize("size", [1.0, 6.0, 96.0, 1536.0, 28672.0])
@pytest.mark.parametrize("sign", [1, -1])
def test_feature_weights_of_a_step_sum_to_one(gpu, D, g, size, sign):
    """The weights that a step books in the feature planes are a softmax whatever the size of the logits (here 1 to 1e10): a single pair has exactly 1,
    the weights of a query sum to 1."""
    fk = gpu
    rows, n, T = 16, 300, 4
    print(f"feature weights D={D} g={g} size={size} sign={sign}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(g)
    mk = lambda *s: (size * torch.randn(s, generator=gen, device="cuda")).to(torch.bfloat16)   # noqa: E731
    desc = fk.CacheDesc(rows, g, 1, D, n + T, "bf16")
    K, V, q, k, v = mk(rows, 1, n + T, D), mk(rows, 1, n + T, D), mk(T, rows, g, D), mk(T, rows, 1, D), mk(T, rows, 1, D)
    ln = torch.full((rows, 1), n, dtype=torch.int32, device="cuda")
    ln[0], ln[1], ln[2] = 0, 31, 255
    _, F = steps_and_window(fk, desc, q, K, V, ln, k, v, sign * D ** -0.5, feat=True)
    live = torch.arange(n + T, device="cuda")[None, :] < ln + T
    booked = (F[:, 0, 3, :, :g].double() * live[:, :, None]).sum(1)
    assert bool(((booked - T).abs() <= T * FEAT_SUM).all()), f"sums off by {(booked - T).abs().max().item():.3g}"
    one = fk.new_feat(desc)
    zero = torch.zeros((rows, 1), dtype=torch.int32, device="cuda")
    out = torch.zeros_like(q[0])
    fk.fk_decode_step_feat(desc, q[0], K, V, torch.zeros((rows, 1, n + T), dtype=torch.int32, device="cuda"), zero, k[0], v[0],
                           torch.zeros(rows, dtype=torch.int32, device="cuda"), 1, sign * D ** -0.5, one, 0, T, out, fk.new_feat_workspace(desc))
    assert bool((one[:, 0, 3, 0, :g] == 1).all()) and torch.equal(out, v[0].expand(rows, g, D))
