"""Decode steps at the edges of the split rule and of the head_dim 64 tiles, against the oracle; the bits of head_dim 64 weights."""
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


# dtype, D, KV heads, group, row length before the step: one split up to 512 keys (bf16), splits of 256 and more above, at most sixteen
# below 512 keys each; fp32: eight splits up to 1024 keys; tiles of 32 keys with 1 or 31 in the last one
CASES = [("bf16", 64, 2, g, n) for g, n in ((1, 30), (2, 31), (3, 32), (4, 511), (5, 512), (6, 513), (7, 767), (8, 1500))]
CASES += [("bf16", 64, 1, 4, 8192), ("bf16", 64, 1, 4, 9000), ("bf16", 128, 1, 4, 8300), ("bf16", 128, 1, 8, 512), ("bf16", 128, 2, 5, 513),
          ("bf16", 64, 40, 2, 600), ("f32", 64, 2, 4, 63), ("f32", 64, 2, 7, 64), ("f32", 128, 1, 4, 300), ("f32", 64, 1, 3, 1024), ("f32", 64, 1, 4, 1060)]
# head_dim 128, cold: one split up to 256 keys, then splits of 96, at most eight
CASES += [("bf16", 128, 16, g, n) for g, n in ((4, 254), (4, 256), (7, 287), (2, 564), (1, 1500))] + [("bf16", 128, 2, 4, 256), ("bf16", 128, 1, 8, 766)]


@pytest.mark.parametrize("dtype,D,H,g,n", CASES)
@pytest.mark.parametrize("cold", [False, True])
def test_step_at_split_and_tile_edges(gpu, ora, dtype, D, H, g, n, cold):
    import paper_2602_03203_amd as fk
    print(f"step {dtype} D={D} Hkv={H} g={g} n={n} cold={cold}", flush=True)
    cap = n + 3
    c = random_cache(ora, 500 + n, dtype, 2, H, cap, D, lens=[n, n // 2])
    dev = gpu.DevCache(c, H * g)
    dev.desc.cold = cold
    ws = fk.new_attn_workspace(dev.desc)
    for t in range(2):
        q, k, v = (random_q(s + t, dtype, 2, h, D) for s, h in ((11, H * g), (21, H), (31, H)))
        pos = np.array([9000 + t, 8000 + t], np.int32)
        ora.append(c, k, v, pos)
        fk.fk_decode_step(dev.desc, gpu.to_dev(q), dev.K, dev.V, dev.pos, dev.len, gpu.to_dev(k), gpu.to_dev(v), gpu.to_dev(pos), n + 1 + t,
                          0.2, dev.out, ws)
        gpu.assert_attn_close(gpu.out_to_f64(dev.out), ora.decode_attn(c, q, 0.2), dtype, f"step {t}")
    host = dev.host(ora)
    assert np.array_equal(host.K, c.K) and np.array_equal(host.V, c.V) and np.array_equal(host.pos, c.pos) and np.array_equal(host.len, c.len)


@pytest.mark.parametrize("D,B,cap,small", [(128, 50, 5400, 3000), (64, 64, 8300, 4000), (64, 64, 8300, 8100)])
def test_rows_taken_by_length_give_the_same_bits(gpu, D, B, cap, small):
    """Many rows and 1 GB of keys and values by the length hint: workgroups take the rows from the longest to the shortest.  A
    smaller hint keeps the plain order and must change nothing: outputs, appended rows, lengths (full, empty, equal ones).  Some
    rows are held against plain sums."""
    import paper_2602_03203_amd as fk
    H, g = 8, 2
    desc = fk.CacheDesc(B, H * g, H, D, cap, "bf16")
    gen = torch.Generator(device="cuda").manual_seed(8)
    mk = lambda *s: torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16)   # noqa: E731
    K0, V0, q, k, v = mk(B, H, cap, D), mk(B, H, cap, D), mk(2, B, H * g, D), mk(2, B, H, D), mk(2, B, H, D)
    lens = torch.randint(0, cap + 1, (B, H), generator=gen, device="cuda", dtype=torch.int32)
    lens[0, 0], lens[1, :4], lens[2] = 0, cap, 77
    pn = torch.arange(2 * B, dtype=torch.int32, device="cuda").reshape(2, B)
    res = []
    for hint in (cap, small):
        K, V, ln, pos, ws = K0.clone(), V0.clone(), lens.clone(), torch.zeros((B, H, cap), dtype=torch.int32, device="cuda"), fk.new_attn_workspace(desc)
        out = torch.zeros_like(q)
        for t in range(2):
            fk.fk_decode_step(desc, q[t], K, V, pos, ln, k[t], v[t], pn[t], hint, 0.1, out[t], ws)
        only = torch.zeros_like(q[0])
        fk.fk_decode_attn(desc, q[0], K, V, ln, hint, 0.1, only, ws)
        assert int(ws[:4 * B * H].view(torch.int32).abs().max()) == 0
        res.append((out, only, ln, pos, K, V))
    assert torch.equal(res[0][2], torch.clamp(lens + 2, max=cap))
    for a, b in zip(*res):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    (_, only, ln, _, K, V), order = res[0], lens.flatten().argsort().tolist()
    for r in [order[i] for i in (1, 2, 3, B * H // 4, B * H // 2, B * H - 7, B * H - 6, B * H - 1)] + [17, 18]:
        b, h = divmod(r, H)
        n = int(ln[b, h])
        z = 0.1 * (q[0, b, h * g:(h + 1) * g].double() @ K[b, h, :n].double().T)
        ref = torch.softmax(z, 1) @ V[b, h, :n].double()
        gpu.assert_attn_close(gpu.out_to_f64(only)[b, h * g:(h + 1) * g], ref.cpu().numpy(), "bf16", f"row {r} of {n} pairs")


@pytest.mark.parametrize("g", [1, 4, 5, 8])
@pytest.mark.parametrize("features", [False, True])
def test_head_dim_64_weights_keep_their_24_bits(gpu, g, features):
    """Four pairs a row: one of weight w and value M, three of weight 1 whose values (bf16 each) add up to -w M, the whole of it.  What is
    left of the sum is M times the error of w.  Derived: a logit of at most 1 is rounded twice (2^-24 of 1.44 each), exp2f is good to
    2^-23 and the sum to 2^-23 of M, below 2^-21 M together; a weight of 16 bits is off by up to 2^-17."""
    import paper_2602_03203_amd as fk
    B, D, M = 256, 64, 2.0 ** 20
    gen = torch.Generator(device="cuda").manual_seed(2)
    desc = fk.CacheDesc(B, g, 1, D, 8, "bf16")
    K, V = torch.zeros((B, 1, 8, D), dtype=torch.bfloat16, device="cuda"), torch.zeros((B, 1, 8, D), dtype=torch.bfloat16, device="cuda")
    q = torch.randn((B, 1, D), generator=gen, device="cuda").to(torch.bfloat16)
    k = torch.randn((B, 1, D), generator=gen, device="cuda").to(torch.bfloat16)
    z = (q.double() * k.double()).sum(2, keepdim=True)
    k = torch.where(z > 0, -k, k)                                   # logits <= 0
    scale = (1.0 / z.abs().amax()).item()                           # the largest is -1
    scale = torch.tensor(scale, dtype=torch.float32).item()
    w = torch.exp((q.double() * k.double()).sum(2) * scale)         # [B][1]
    rest = w * M
    for slot in range(3):
        v = rest.to(torch.bfloat16)
        V[:, :, slot, :] = -v[:, :, None]
        rest = rest - v.double()
    qg = q.expand(B, g, D).contiguous()
    ln, pos = torch.full((B, 1), 3, dtype=torch.int32, device="cuda"), torch.zeros((B, 1, 8), dtype=torch.int32, device="cuda")
    vn, pn, out = torch.full((B, 1, D), M, dtype=torch.bfloat16, device="cuda"), torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros_like(qg)
    if features:
        fk.fk_decode_step_feat(desc, qg, K, V, pos, ln, k, vn, pn, 4, scale, fk.new_feat(desc), 0, 4, out, fk.new_feat_workspace(desc))
    else:
        fk.fk_decode_step(desc, qg, K, V, pos, ln, k, vn, pn, 4, scale, out, fk.new_attn_workspace(desc))
    off = (out.double() * (3.0 + w[:, :, None]) - rest[:, :, None]).abs() / M
    assert off.max() < 2.0 ** -21, f"weights off by 2^{torch.log2(off.max()).item():.1f}"


# rows, group, head_dim, capacity (the length hint): a workgroup per query head up to a length by head_dim, rows (up to 15, 63, 256) and heads, 256
# workgroups, and, where the rows are no multiple of eight, copies of K and V that fit the L2s; both sides of these lines
BY_HEAD = [(2, 4, 64, 300), (2, 1, 64, 390), (2, 1, 64, 391), (8, 2, 128, 300), (8, 2, 128, 301), (3, 8, 64, 520), (32, 8, 128, 140), (33, 8, 128, 140),
           (5, 3, 128, 500), (21, 4, 128, 390), (21, 4, 128, 391), (16, 5, 64, 257), (1, 7, 128, 9), (256, 1, 64, 70),
           (8, 2, 128, 140), (8, 2, 128, 141), (16, 1, 128, 250), (16, 1, 128, 251), (64, 4, 128, 900), (64, 4, 64, 810), (15, 3, 64, 340), (128, 2, 64, 661)]


@pytest.mark.parametrize("rows,g,D,cap", BY_HEAD)
def test_fp32_steps_by_query_head(gpu, rows, g, D, cap):
    """Three steps of rows at the edges of the wavefronts' rounds (16 wavefronts of 16 or 8 pairs), empty and full ones among them, with the
    tolerance of the other fp32 steps; lengths, new pairs and counters as they must be."""
    import paper_2602_03203_amd as fk
    print(f"fp32 by head rows={rows} g={g} D={D} cap={cap}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(rows + g + cap)
    mk = lambda *s: torch.randn(s, generator=gen, device="cuda")   # noqa: E731
    desc = fk.CacheDesc(rows, g, 1, D, cap, "f32")
    K, V, q, k, v = mk(rows, 1, cap, D), mk(rows, 1, cap, D), mk(3, rows, g, D), mk(3, rows, 1, D), mk(3, rows, 1, D)
    edges = [0, cap, cap - 1, cap - 2, 1, 15, 16, 127, 128, 255, 256]
    ln = torch.tensor([min(edges[r % len(edges)], cap) for r in range(rows)], dtype=torch.int32, device="cuda").reshape(rows, 1)
    pos, pn = torch.zeros((rows, 1, cap), dtype=torch.int32, device="cuda"), torch.arange(3 * rows, dtype=torch.int32, device="cuda").reshape(3, rows) + 7
    ws, out, K0, V0, n0 = fk.new_attn_workspace(desc), torch.zeros_like(q), K.clone(), V.clone(), ln[:, 0].tolist()
    K[:, :, cap // 2 + 1:][torch.arange(cap // 2 + 1, cap, device="cuda")[None, None, :] >= ln[:, :, None]] = float("nan")   # what is not live is not used
    V.masked_fill_(torch.isnan(K), float("nan"))
    for t in range(3):
        fk.fk_decode_step(desc, q[t], K, V, pos, ln, k[t], v[t], pn[t], cap, 0.3, out[t], ws)
    assert int(ws[:4 * rows].view(torch.int32).abs().max()) == 0
    for r in range(rows):
        n = n0[r]
        for t in range(3):
            if n < cap:
                K0[r, 0, n], V0[r, 0, n] = k[t, r, 0], v[t, r, 0]
                assert int(pos[r, 0, n]) == int(pn[t, r])
                n += 1
            p = torch.softmax(0.3 * (q[t, r].double() @ K0[r, 0, :n].double().T), 1)
            gpu.assert_attn_close(out[t, r].double().cpu().numpy(), (p @ V0[r, 0, :n].double()).cpu().numpy(), "f32", f"row {r} of {n} pairs, step {t}")
        assert int(ln[r, 0]) == n and torch.equal(K[r, 0, :n], K0[r, 0, :n]) and torch.equal(V[r, 0, :n], V0[r, 0, :n])
