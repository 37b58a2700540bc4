"""fk_decode_window and fk_decode_window_feat on a whole window at once: bit for bit the single steps over the splits, tile walks and
workgroup shapes of the launch rules, the edges of the tiles, rows that fill up inside the window, and calls whose buffers order the steps."""
import numpy as np
import pytest
import torch

from util import random_cache, random_q

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util
    import paper_2602_03203_amd as fk
    fk.lib()
    return gpu_util


def oracle_window(ora, c, q, k, v, pos, scale):
    """The steps one by one on the oracle, rows as one-head sequences; c is advanced."""
    T, Bt, Hq, D = q.shape
    H = k.shape[2]
    g = Hq // H
    out = np.empty(q.shape, np.float64)
    for t in range(T):
        for r in np.nonzero(c.len < c.shape[2])[0]:
            sub = ora.Cache(c.dtype, c.K[r:r + 1], c.V[r:r + 1], c.pos[r:r + 1], c.len[r:r + 1])
            ora.append(sub, k[t].reshape(Bt * H, 1, D)[r:r + 1], v[t].reshape(Bt * H, 1, D)[r:r + 1], pos[t, r // H:r // H + 1])
        out[t] = ora.decode_attn(c, q[t].reshape(Bt * H, g, D), scale).reshape(Bt, Hq, D)
    return out


# D, batch, KV heads, group, capacity, steps, row lengths (cycled over the rows), scale
WINDOWS = [
    (128, 16, 8, 4, 200, 66, [60, 0, 199, 131, 64, 63], 0.09),    # two groups of steps a workgroup, a ragged last one; full rows
    (64, 16, 16, 8, 140, 5, [64, 1, 0, 127, 139], 0.125),          # head_dim 64, two steps to a group
    (128, 16, 8, 7, 300, 33, [128, 255, 40], 0.3),                 # group of 7: two rows of a matrix product unused
    (64, 16, 8, 5, 260, 40, [100, 259, 0], 0.2),                   # group of 5, head_dim 64
    (128, 16, 8, 3, 300, 40, [128, 0, 290], 0.09),                 # one group of steps a workgroup
    (64, 16, 8, 1, 600, 70, [500, 10], 0.4),                       # one head per group: sixteen steps in a product
    (128, 1, 2, 4, 700, 17, [530, 690], 0.09),                     # few rows, split
    (64, 2, 1, 8, 400, 2, [399, 128], 0.125),                      # two steps, one row full after the first
    (128, 2, 2, 4, 150, 9, [140, 3, 31, 32], -0.09),               # a negative scale
    (64, 1, 2, 2, 90, 12, [50, 0], 0.0),                           # scale 0: plain means
]


@pytest.mark.parametrize("D,Bt,H,g,cap,T,lens,scale", WINDOWS)
def test_window_at_once_matches_oracle(gpu, ora, D, Bt, H, g, cap, T, lens, scale):
    import paper_2602_03203_amd as fk
    print(f"window case D={D} batch={Bt} Hkv={H} g={g} cap={cap} T={T} scale={scale}", flush=True)
    R = Bt * H
    ln = np.array([lens[r % len(lens)] for r in range(R)], np.int32)
    c = random_cache(ora, 100 + D + T, "bf16", R, 1, cap, D, lens=ln)
    q = random_q(101, "bf16", T, Bt * H * g, D).reshape(T, Bt, H * g, D)
    k, v = (random_q(s, "bf16", T, R, D).reshape(T, Bt, H, D) for s in (102, 103))
    pos = (10 ** 6 + np.arange(T)[:, None] + 1000 * np.arange(Bt)[None, :]).astype(np.int32)
    desc = fk.CacheDesc(Bt, H * g, H, D, cap, "bf16")
    K, V = gpu.to_dev(c.K.reshape(Bt, H, cap, D)), gpu.to_dev(c.V.reshape(Bt, H, cap, D))
    dpos, dlen, ws = gpu.to_dev(c.pos.reshape(Bt, H, cap)), gpu.to_dev(ln.reshape(Bt, H)), fk.new_attn_workspace(desc)
    out = torch.zeros((T, Bt, H * g, D), dtype=torch.bfloat16, device="cuda")
    fk.fk_decode_window(desc, gpu.to_dev(q), K, V, dpos, dlen, gpu.to_dev(k), gpu.to_dev(v), gpu.to_dev(pos), T,
                        min(int(ln.max()) + 1, cap), scale, out, ws)
    ref = oracle_window(ora, c, q, k, v, pos, scale)
    gpu.assert_attn_close(gpu.out_to_f64(out), ref, "bf16", "window")
    assert np.array_equal(gpu.to_host(dlen).reshape(-1), c.len) and np.array_equal(gpu.to_host(dpos).reshape(c.pos.shape), c.pos)
    assert np.array_equal(gpu.to_host(K).reshape(c.K.shape), c.K) and np.array_equal(gpu.to_host(V).reshape(c.V.shape), c.V)
    assert int(ws[:4 * R].view(torch.int32).abs().max()) == 0   # the arrival counters are back at zero


def window_and_steps(gpu, fk, desc, args, T, ml, scale, feat=None, c0=0, L=0):
    """Final buffers after one window call and after the single steps."""
    res = []
    for window in (True, False):
        q, K, V, pos, ln, k, v, pn = (a.clone() for a in args)
        out = torch.zeros_like(q)
        f = None if feat is None else feat.clone()
        ws = fk.new_attn_workspace(desc) if feat is None else fk.new_feat_workspace(desc).fill_(0xA5)   # (needs no initialisation)
        counters = (desc.batch * desc.n_kv_heads * 4 + 255) // 256 * 256
        if feat is None:
            ws[counters:] = 0xA5
        for t in range(0 if window else T):
            m = min(ml + t, desc.capacity)
            if feat is None:
                fk.fk_decode_step(desc, q[t], K, V, pos, ln, k[t], v[t], pn[t], m, scale, out[t], ws)
            else:
                fk.fk_decode_step_feat(desc, q[t], K, V, pos, ln, k[t], v[t], pn[t], m, scale, f, c0 + t, L, out[t], ws)
        if window and feat is None:
            fk.fk_decode_window(desc, q, K, V, pos, ln, k, v, pn, T, ml, scale, out, ws)
            assert bool((ws[counters:] == 0xA5).all())   # at once: single steps of split rows leave their records there
            assert int(ws[:counters].max()) == 0
        elif window:
            fk.fk_decode_window_feat(desc, q, K, V, pos, ln, k, v, pn, T, ml, scale, f, c0, L, out, ws)
        torch.cuda.synchronize()
        res.append((out, K, V, pos, ln) + (() if f is None else (f,)))
    return res


def device_args(desc, T, lens, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    mk = lambda *shape: torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)   # noqa: E731
    B, H, cap, D = desc.batch, desc.n_kv_heads, desc.capacity, desc.head_dim
    ln = torch.tensor([lens[r % len(lens)] for r in range(B * H)], dtype=torch.int32, device="cuda").reshape(B, H)
    pos = torch.arange(cap, dtype=torch.int32, device="cuda").expand(B, H, cap).contiguous()
    pn = torch.arange(T * B, dtype=torch.int32, device="cuda").reshape(T, B) + 5000
    return mk(T, B, desc.n_q_heads, D), mk(B, H, cap, D), mk(B, H, cap, D), pos, ln, mk(T, B, H, D), mk(T, B, H, D), pn


# D, batch, KV heads, group, capacity, steps, row lengths, length hint, cold, scale.  Splits: how many and how long follows from the hint
# of every step, so it changes inside a window (1536 pairs: six to seven splits); long ones are walked from another tile in every
# row (2 x 2112 pairs); more than 64 take the merge in batches.
BITS = [
    (128, 16, 8, 4, 200, 66, [60, 0, 199, 131, 64, 63], 200, False, 0.09),
    (64, 32, 8, 8, 140, 5, [64, 1, 0, 127, 139], 140, False, 0.125),
    (128, 16, 8, 7, 300, 33, [128, 255, 40], 256, False, -0.3),
    (64, 1, 8, 5, 500, 40, [440, 259, 0], 441, False, 0.2),
    (128, 2, 4, 4, 1700, 100, [1500, 1400, 3], 1501, False, 0.09),
    (64, 2, 4, 4, 1700, 100, [1500, 1400, 3], 1501, False, 0.0),
    (128, 3, 2, 3, 700, 50, [500, 3, 0], 501, False, 0.3),
    (64, 8, 8, 1, 900, 40, [880, 31, 899], 881, True, 0.3),
    (128, 4, 8, 3, 700, 30, [600, 699, 0], 601, True, 0.3),
    (128, 1, 4, 4, 700, 40, [480, 699, 250], 481, True, 0.1),     # few cold rows: six to seven splits of 96
    (128, 1, 3, 8, 700, 50, [680, 3, 699], 600, False, 0.1),
    (128, 8, 8, 2, 4300, 40, [4200, 100, 4095], 4201, False, 0.09),
    (64, 2, 8, 6, 40000, 30, [39000, 100, 32767], 39001, True, 0.09),
    (128, 1, 1, 4, 66000, 90, [65950], 65951, False, 0.09),
    (64, 1, 1, 2, 66000, 90, [65930], 65951, False, 0.09),
]


@pytest.mark.parametrize("D,Bt,H,g,cap,T,lens,hint,cold,scale", BITS)
def test_window_equals_the_single_steps_bit_for_bit(gpu, D, Bt, H, g, cap, T, lens, hint, cold, scale):
    import paper_2602_03203_amd as fk
    print(f"window bits D={D} batch={Bt} Hkv={H} g={g} cap={cap} T={T} lens={lens} cold={cold}", flush=True)
    desc = fk.CacheDesc(Bt, H * g, H, D, cap, "bf16", cold=cold)
    a, b = window_and_steps(gpu, fk, desc, device_args(desc, T, lens, D + T), T, hint, scale)
    for x, y in zip(a, b):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))


@pytest.mark.parametrize("g", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("T,c0,L,lens,cap", [(37, 0, 37, [300, 0, 281, 31], 333), (9, 60, 128, [64, 255, 1], 300), (64, 0, 64, [700, 10], 800),
                                             (5, 3, 200, [9, 12], 16)])
def test_window_with_features_equals_the_single_steps_bit_for_bit(gpu, g, T, c0, L, lens, cap):
    import paper_2602_03203_amd as fk
    print(f"feature window g={g} T={T} chunk {c0}/{L} lens={lens} cap={cap}", flush=True)
    desc = fk.CacheDesc(3, 2 * g, 2, 128, cap, "bf16")
    args = device_args(desc, T, lens, 7 * g + T)
    feat = torch.rand((3, 2, 6, cap, fk.feat_heads(desc)), device="cuda")
    a, b = window_and_steps(gpu, fk, desc, args, T, min(max(lens) + 1, cap), 0.2, feat, c0, L)
    for x, y in zip(a, b):
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8))


@pytest.mark.parametrize("D,features", [(128, False), (128, True), (64, False)])
def test_window_keeps_a_later_steps_infinities_from_the_earlier_ones(gpu, D, features):
    """A value row of step 5 that holds an infinity and a NaN reaches the outputs from step 5 on, and no other, in a window as in the
    single steps."""
    import paper_2602_03203_amd as fk
    T = 12
    desc = fk.CacheDesc(2, 8, 2, D, 128, "bf16")
    args = list(device_args(desc, T, [70, 33], 3))
    clean = [a.clone() for a in args]
    args[6][5, 1, 0, 17], args[6][5, 1, 0, 40] = float("inf"), float("nan")
    clean[6][5, 1, 0, 17], clean[6][5, 1, 0, 40] = 0.0, 0.0
    feat = torch.zeros((2, 2, 6, 128, 4), device="cuda") if features else None
    got, steps = window_and_steps(gpu, fk, desc, args, T, 71, 0.1, feat, 0, 32)
    for a, b in zip(got, steps):
        assert torch.equal(a.isnan(), b.isnan()) and torch.equal(torch.nan_to_num(a.double(), 0.5), torch.nan_to_num(b.double(), 0.5))
    ref = window_and_steps(gpu, fk, desc, clean, T, 71, 0.1, feat, 0, 32)[0]
    o, r = got[0].float(), ref[0].float()
    assert torch.isposinf(o[5:, 1, :4, 17]).all() and torch.isnan(o[5:, 1, :4, 40]).all()
    o[5:, 1, :4, 17], o[5:, 1, :4, 40] = r[5:, 1, :4, 17], r[5:, 1, :4, 40]
    assert torch.equal(o, r)
    if features:
        assert torch.equal(got[5], ref[5])


def test_window_whose_buffers_order_the_steps_runs_step_by_step(gpu):
    """One step's output is the next one's query (a buffer that is out_seq and, one step on, q_seq): the steps in their order."""
    import paper_2602_03203_amd as fk
    T, D = 6, 128
    desc = fk.CacheDesc(2, 8, 2, D, 64, "bf16")
    q, K, V, pos, ln, k, v, pn = device_args(desc, T, [20, 31], 9)
    res = []
    for window in (True, False):
        Kx, Vx, px, lx, ws = K.clone(), V.clone(), pos.clone(), ln.clone(), fk.new_attn_workspace(desc)
        buf = torch.zeros((T + 1, 2, 8, D), dtype=torch.bfloat16, device="cuda")
        buf[0] = q[0]
        if window:
            fk.fk_decode_window(desc, buf[:T], Kx, Vx, px, lx, k, v, pn, T, 32, 0.2, buf[1:], ws)
        else:
            for t in range(T):
                fk.fk_decode_step(desc, buf[t], Kx, Vx, px, lx, k[t], v[t], pn[t], 32 + t, 0.2, buf[t + 1], ws)
        res.append((buf, Kx, Vx, px, lx))
    for a, b in zip(*res):
        assert torch.equal(a, b)
