"""uad_set_prefix_kv from every kind of source: the same values handed over as
device fp32 / bf16 (aligned or offset by one element), host fp32 / bf16, and a
prefix too long for one staging run give the same step bit for bit, and that
step matches the oracle.  Bars as for the other parity tests."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as O
import paper_2609_37772_amd as U
import uad_workloads as W
from tests.harness import log, rel_err

pytestmark = pytest.mark.gpu


def offset_by_one(a):
    """The same device tensor, its data one element past a 16-byte boundary."""
    buf = torch.empty(a.numel() + 1, dtype=a.dtype, device="cuda")
    out = buf[1:].view(a.shape)
    out.copy_(a)
    assert out.data_ptr() % 16 != 0
    return out


# head dim, KV heads, batch, chunk, prefix: ragged 32-key blocks, one key, whole
# blocks, no prefix, and 9000 keys x 2 heads x 256 fp32 (over half the 32 MiB
# staging workspace: an environment goes up in runs of 32-key blocks); 520 heads:
# one fp32 block exceeds the workspace (a buffer of the call's own)
@pytest.mark.parametrize("hd,hkv,B,H,P", [(64, 4, 2, 5, 33), (128, 2, 3, 16, 64), (256, 1, 2, 7, 1), (64, 2, 1, 3, 0),
                                           (256, 2, 1, 4, 9000), (256, 520, 1, 3, 33)])
def test_prefix_sources_agree(gpu, hd, hkv, B, H, P):
    shape = W.ModelShape(2, 128, max(4, hkv), hkv, hd, 256, 7)
    wl = dataclasses.replace(W.get_workload("tiny"), shape=shape, batch=B, chunk=H, prefix=P)
    weights = W.make_weights(wl)
    g = np.random.default_rng(hd + P)
    k, v = (g.standard_normal((2, B, P, hkv, hd), dtype=np.float32) for _ in range(2))
    k.reshape(-1)[::7] = np.float32(1.00390625)  # half way between two bf16 values: ties to even
    kb, vb = W.round_to_bf16(k), W.round_to_bf16(v)
    x0 = np.stack([W.make_noise(wl, b) for b in range(B)])
    t = np.full((B, H), 0.5, np.float32)
    dt = np.full((B, H), -0.1, np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    kd, vd = dev(k), dev(v)
    k16, v16 = dev(kb).to(torch.bfloat16), dev(vb).to(torch.bfloat16)
    sources = {"host fp32": (k, v), "host bf16": (W.bf16_bits(kb), W.bf16_bits(vb))}
    if P:  # an empty device tensor has no address
        sources.update({"device fp32": (kd, vd), "device bf16": (k16, v16)})
        sources["device fp32 offset"] = (offset_by_one(kd), vd)
        sources["device bf16 offset"] = (k16, offset_by_one(v16))
    ex = U.ActionExpert(shape, B + 1, H, P + 40)  # larger than the call: other environments' slots, spare blocks
    try:
        ex.load_weights(weights)
        got = {}
        for name, (ks, vs) in sources.items():
            # a full store first, so that stale keys would show
            ones = torch.ones((2, B + 1, P + 40, hkv, hd), device="cuda")
            ex.set_prefix_kv(ones, ones, B + 1, P + 40)
            ex.set_prefix_kv(ks, vs, B, P)
            x, vel = dev(x0), torch.empty((B, H, 7), device="cuda")
            ex.step(x, dev(t), dev(dt), torch.zeros((B, H), dtype=torch.uint8, device="cuda"), vel)
            ex.synchronize()
            got[name] = (x.cpu().numpy().tobytes(), vel.cpu().numpy())
        first = got["host fp32"]
        for name, (xb, vel) in got.items():
            assert xb == first[0] and vel.tobytes() == first[1].tobytes(), name
        m = O.build_model(shape, weights, [kb[:, b] for b in range(B)], [vb[:, b] for b in range(B)])
        e = rel_err(first[1], O.velocity(m, x0, t))
        log(f"[prefix hd={hd} Hkv={hkv} B={B} P={P}] {len(got)} sources bit-identical, velocity rel err {e:.2e}")
        assert e <= 2e-2
    finally:
        ex.close()
