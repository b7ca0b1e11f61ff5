"""Batched steps of the adaptive-norm expert (over 256 token rows): the
modulations of the distinct flow times only, the norms as passes of their own.
The row counts on either side of the bound, all tokens at one time, a few times in an irregular order, every token its own
(272 rows), more distinct times than the class table takes (1120 rows), widths
that are not multiples of 64 or 256, and ragged last row tiles; sampled
environments against the oracle, the no-allocation step bit for bit.  Bars as
for the other parity tests."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as O
import paper_2609_37772_amd as U
import uad_workloads as W
from paper_2609_37772_amd import _binding as B_
from tests.harness import log, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,B,H,times", [
    (256, 16, 16, 3), (256, 15, 17, 3), (256, 17, 16, 1), (256, 17, 16, 272), (96, 19, 14, 5), (320, 70, 16, 1120), (512, 65, 17, 9), (512, 65, 17, 1024),
])
def test_batched_times(gpu, d, B, H, times):
    shape = W.ModelShape(2, d, 4, 2, 64, 2 * d, 7, conditioning="adarms")
    wl = dataclasses.replace(W.get_workload("tiny_adarms"), shape=shape, batch=B, chunk=H, prefix=40)
    weights = W.make_weights(wl)
    g = np.random.default_rng(d + times)
    k, v = (W.round_to_bf16(g.standard_normal((2, B, 40, 2, 64), dtype=np.float32)) for _ in range(2))
    x0 = np.stack([W.make_noise(wl, b) for b in range(B)])
    t = (((np.arange(B * H, dtype=np.int64) * 7919) % times + 1) / np.float32(times)).astype(np.float32).reshape(B, H)
    assert len(np.unique(t)) == times
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ex = U.ActionExpert(shape, B, H, 40)
    try:
        ex.load_weights(weights)
        ex.set_prefix_kv(W.bf16_bits(k), W.bf16_bits(v), B, 40)
        got = []
        for fn in (B_.uad_denoise_step, B_.uad_denoise_step, B_.uad_denoise_step_static):
            x, vel = dev(x0), torch.empty((B, H, 7), device="cuda")
            fn(ex.ctx, x, dev(t), torch.full((B, H), -0.1, device="cuda"),
               torch.zeros((B, H), dtype=torch.uint8, device="cuda"), vel)
            ex.synchronize()
            got.append(vel.cpu().numpy())
        assert got[0].tobytes() == got[1].tobytes() == got[2].tobytes()
        for b in (0, B // 2, B - 1):
            m = O.build_model(shape, weights, [k[:, b]], [v[:, b]])
            e = rel_err(got[0][b], O.velocity(m, x0[b:b + 1], t[b:b + 1])[0])
            log(f"[adarms d={d} rows={B * H} times={times}] env {b}: velocity rel err {e:.2e}")
            assert e <= 2e-2
    finally:
        ex.close()
