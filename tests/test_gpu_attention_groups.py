"""Attention with two key groups per workgroup (long splits on a grid of at most
one workgroup per CU): odd and even block counts, a partly masked last block, a
last split of one block (its second group has none), one split and several, at
each head dim.  Step velocities of sampled environments against the oracle, and
a repeated step bit for bit.  Bar as for the other parity tests."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as O
import paper_2609_37772_amd as U
import uad_workloads as W
from tests.harness import log, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,heads,hkv,B,H,keys", [
    (256, 2, 1, 130, 16, 5 * 32),        # one split of 5 blocks: groups of 3 and 2
    (256, 2, 1, 130, 16, 6 * 32 - 31),   # 6 blocks, one key in the last
    (128, 4, 2, 70, 9, 9 * 32 - 5),      # 9 blocks of 128-wide heads
    (64, 4, 4, 40, 20, 10 * 32 - 1),     # 10 blocks of 64-wide heads
    (256, 2, 1, 40, 16, 25 * 32 - 7),    # five splits of 6 blocks, the last of 1
    (128, 2, 1, 30, 16, 70 * 32 - 3),    # several long splits of 128-wide heads
])
def test_two_key_groups(gpu, hd, heads, hkv, B, H, keys):
    shape = W.ModelShape(2, 128, heads, hkv, hd, 256, 7)
    wl = dataclasses.replace(W.get_workload("tiny"), shape=shape, batch=B, chunk=H, prefix=keys - H)
    weights = W.make_weights(wl)
    g = np.random.default_rng(keys)
    k, v = (W.round_to_bf16(g.standard_normal((2, B, keys - H, hkv, hd), dtype=np.float32)) for _ in range(2))
    x0 = np.stack([W.make_noise(wl, b) for b in range(B)])
    t = np.full((B, H), 0.5, np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ex = U.ActionExpert(shape, B, H, keys - H)
    try:
        ex.load_weights(weights)
        ex.set_prefix_kv(W.bf16_bits(k), W.bf16_bits(v), B, keys - H)
        vels = []
        for _ in range(2):
            x, vel = dev(x0), torch.empty((B, H, 7), device="cuda")
            ex.step(x, dev(t), torch.full((B, H), -0.1, device="cuda"),
                    torch.zeros((B, H), dtype=torch.uint8, device="cuda"), vel)
            ex.synchronize()
            vels.append(vel.cpu().numpy())
        assert vels[0].tobytes() == vels[1].tobytes()
        for b in (0, B // 2, B - 1):
            m = O.build_model(shape, weights, [k[:, b]], [v[:, b]])
            e = rel_err(vels[0][b], O.velocity(m, x0[b:b + 1], t[b:b + 1])[0])
            log(f"[key groups hd={hd} B={B} keys={keys}] env {b}: velocity rel err {e:.2e}")
            assert e <= 2e-2
    finally:
        ex.close()
