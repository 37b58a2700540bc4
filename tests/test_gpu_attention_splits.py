"""Decode steps at the edges of the split rule and of the head_dim 64 tiles, against the oracle."""
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
