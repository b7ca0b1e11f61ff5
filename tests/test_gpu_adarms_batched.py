"""Batched steps of the adaptive-norm expert (256 token rows and more): the
modulations of the distinct flow times only, the norms as passes of their own.
The row counts on either side of the bound, all tokens at one time, a few times in
an irregular order, every token its own (272 rows), more distinct times than the class table takes (1120 rows), widths
that are not multiples of 64 or 256, and ragged last row tiles; sampled
environments against the oracle, the no-allocation step bit for bit.  Then the
experts' own widths on each kernel of the products (tests/test_routes.py has the
rules): the row count known on the device only in the register-streamed kernel,
whole and in k-halves, and the gates by class in the ring and streamed residual
epilogues.  And a schedule of 256 rows on either side of the rule for exactly that
many: a narrow expert by token, conditioned once for the schedule, and a wider one
by class.  The widths from 1024 up have the bar of the other parity tests.  The
small ones need a closer one: with modulations of 0.02 sqrt(d) their layers move
the velocity so little that a token with its neighbour's flow time shows only
2.6e-3 (oracle, 96 wide) to 6.7e-2; the errors are 6e-5 to 3.6e-4."""
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
SMALL_BAR, BAR = 1.5e-3, 2e-2


def _check(shape, B, H, times, label, bar):
    d, P = shape.d_model, 40
    wl = dataclasses.replace(W.get_workload("tiny_adarms"), shape=shape, batch=B, chunk=H, prefix=P)
    weights = W.make_weights(wl)
    g = np.random.default_rng(d + times)
    kv = (shape.n_layers, B, P, shape.n_kv_heads, shape.head_dim)
    k, v = (W.round_to_bf16(g.standard_normal(kv, dtype=np.float32)) for _ in range(2))
    x0 = np.stack([W.make_noise(wl, b) for b in range(B)])
    t = (((np.arange(B * H, dtype=np.int64) * 7919) % times + 1) / np.float32(times)).astype(np.float32).reshape(B, H)
    assert len(np.unique(t)) == times
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ex = U.ActionExpert(shape, B, H, P)
    try:
        ex.load_weights(weights)
        ex.set_prefix_kv(W.bf16_bits(k), W.bf16_bits(v), B, P)
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
            log(f"[adarms {label} d={d} rows={B * H} times={times}] env {b}: velocity rel err {e:.2e}")
            assert e <= bar
    finally:
        ex.close()


@pytest.mark.parametrize("d,B,H,times", [
    (256, 16, 16, 3), (256, 15, 17, 3), (256, 17, 16, 1), (256, 17, 16, 272), (96, 19, 14, 5),
    (320, 70, 16, 1120), (512, 65, 17, 9), (512, 65, 17, 1024),
])
def test_batched_times(gpu, d, B, H, times):
    _check(W.ModelShape(2, d, 4, 2, 64, 2 * d, 7, conditioning="adarms"), B, H, times, "times", SMALL_BAR)


# width, heads, KV heads, head dim, MLP width, environments, chunk, flow times
WIDE = [
    (1024, 8, 1, 256, 4096, 64, 50, 9),    # 3200 rows: time MLP streamed, O on the 128 x 128 ring, down split there
    (1536, 12, 2, 128, 6144, 11, 128, 5),  # 1408: time MLP and O streamed in k-halves, down split on 128 x 96
    (1536, 4, 2, 64, 2048, 11, 127, 200),  # 1397: O streamed whole (K = 256), ragged; two row panels of times
    (1536, 12, 2, 128, 6144, 16, 128, 3),  # 2048: O on the 128 x 96 ring
]


@pytest.mark.parametrize("d,heads,hkv,hd,F,B,H,times", WIDE)
def test_batched_wide(gpu, d, heads, hkv, hd, F, B, H, times):
    _check(W.ModelShape(2, d, heads, hkv, hd, F, 7, conditioning="adarms"), B, H, times, "wide", BAR)


@pytest.mark.parametrize("d,layers", [(256, 4), (768, 2)])
def test_schedule_at_the_bound(gpu, d, layers):
    shape = W.ModelShape(layers, d, 4, 2, 64, 4 * d, 7, conditioning="adarms")
    _check(shape, 16, 16, 5, "bound", SMALL_BAR)
    B, H, P = 16, 16, 40
    wl = dataclasses.replace(W.get_workload("tiny_adarms"), shape=shape, batch=B, chunk=H, prefix=P)
    weights = W.make_weights(wl)
    g = np.random.default_rng(d)
    k, v = (W.round_to_bf16(g.standard_normal((layers, B, P, 2, 64), dtype=np.float32)) for _ in range(2))
    x0 = np.stack([W.make_noise(wl, b) for b in range(B)]).astype(np.float32)
    bud = np.full((B, H), 5, np.int32)
    bud[:, :3] = 2
    ex = U.ActionExpert(shape, B, H, P)
    try:
        ex.load_weights(weights)
        ex.set_prefix_kv(W.bf16_bits(k), W.bf16_bits(v), B, P)
        n, t, dt, mask = ex.schedule_tables(bud)
        got = []
        for _ in range(2):
            x = torch.from_numpy(x0).cuda()
            rel = torch.zeros_like(x)
            ex.schedule(x, t, dt, mask, rel)
            torch.cuda.synchronize()
            got.append(rel.cpu().numpy())
        assert got[0].tobytes() == got[1].tobytes()
        for b in (0, B - 1):
            r = O.denoise_schedule(O.build_model(shape, weights, [k[:, b]], [v[:, b]]), x0[b:b + 1], bud[b:b + 1])
            e = rel_err(got[0][b], r["released"][0])
            log(f"[adarms schedule d={d}] env {b}: released rel err {e:.2e}")
            assert e <= SMALL_BAR
    finally:
        ex.close()
