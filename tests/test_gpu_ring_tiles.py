"""Projection tiles of a few hundred rows, each on ragged row counts: gate/up on
64 x 128 and 128 x 128 ring tiles, QKV on 64 x 64 and 64 x 128, the residual
projections on 64 x 64 whole and split over K two and four ways, and the counts
just past the last bound; and 288 columns, which have no 64 x 64 tiles, so that
a short K splits on 128 x 96 ones.  Step velocities of sampled environments against the
oracle, a repeated step bit for bit.  Bar as for the other parity tests."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as O
import paper_2609_37772_amd as U
import uad_workloads as W
from tests.harness import log, rel_err

pytestmark = pytest.mark.gpu


def _check(shape, B, H):
    P = 45
    wl = dataclasses.replace(W.get_workload("tiny"), shape=shape, batch=B, chunk=H, prefix=P)
    weights = W.make_weights(wl)
    g = np.random.default_rng(B * H)
    k, v = (W.round_to_bf16(g.standard_normal((2, B, P, 1, 256), dtype=np.float32)) for _ in range(2))
    x0 = np.stack([W.make_noise(wl, b) for b in range(B)])
    t = np.full((B, H), 0.5, np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ex = U.ActionExpert(shape, B, H, P)
    try:
        ex.load_weights(weights)
        ex.set_prefix_kv(W.bf16_bits(k), W.bf16_bits(v), B, P)
        vels = []
        for _ in range(4):
            x, vel = dev(x0), torch.empty((B, H, 7), device="cuda")
            ex.step(x, dev(t), torch.full((B, H), -0.1, device="cuda"),
                    torch.zeros((B, H), dtype=torch.uint8, device="cuda"), vel)
            ex.synchronize()
            vels.append(vel.cpu().numpy())
        assert all(v.tobytes() == vels[0].tobytes() for v in vels)
        for b in (0, B // 2, B - 1):
            m = O.build_model(shape, weights, [k[:, b]], [v[:, b]])
            e = rel_err(vels[0][b], O.velocity(m, x0[b:b + 1], t[b:b + 1])[0])
            log(f"[ring tiles rows={B * H}] env {b}: velocity rel err {e:.2e}")
            assert e <= 2e-2
    finally:
        ex.close()


@pytest.mark.parametrize("B,H", [
    (7, 19),   # 133 rows: gate/up 64 x 128, QKV still on the small-M kernel
    (5, 51),   # 255: QKV 64 x 64, the last row tile one short
    (13, 49),  # 637: gate/up 128 x 128, down split four ways over 80 tiles
    (21, 61),  # 1281: O on 64 x 64, down split four ways over 168 tiles
    (31, 51),  # 1581: QKV 64 x 128, down split two ways over 200 tiles
    (33, 53),  # 1749: past the bounds of both
])
def test_ring_tiles(gpu, B, H):
    _check(W.ModelShape(2, 512, 8, 1, 256, 4096, 7), B, H)


def test_split_short_k(gpu):
    """3750 rows x 288 columns, K = 1024: 90 tiles of 128 x 96, split two ways."""
    _check(W.ModelShape(2, 288, 4, 1, 256, 1024, 7), 30, 125)
