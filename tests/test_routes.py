"""The dispatch rules on the CPU: the GPU tests' sizes take the kernels that
those tests name."""
import pytest

from tests import routes as R

D, F, QD, NQKV = 512, 4096, 2048, 2560  # the expert of test_gpu_ring_tiles


@pytest.mark.parametrize("rows,gateup,qkv,o,down", [
    (133, (64, 128), None, None, None),
    (255, (64, 128), (64, 64), None, None),
    (637, (128, 128), (64, 64), None, (64, 64, 4)),
    (1281, (128, 256), (128, 128), (64, 64, 1), (64, 64, 4)),
    (1581, (128, 256), (64, 128), (64, 64, 1), (64, 64, 2)),
    (1749, (128, 256), (128, 128), (64, 64, 1), None),
])
def test_ring_tile_sizes(rows, gateup, qkv, o, down):
    def ring(epi, N, K, q_dim=0):
        r = R.projection(epi, rows, N, K, q_dim=q_dim)
        return r[1:] if r[0] == R.RING else None
    assert (ring(R.GEGLU, 2 * F, D) or (None,) * 2)[:2] == (gateup or (None,) * 2)
    assert (ring(R.QKV, NQKV, D, QD) or (None,) * 2)[:2] == (qkv or (None,) * 2)
    assert (ring(R.RESID, D, QD) or (None,) * 3)[:3] == (o or (None,) * 3)
    assert (ring(R.RESID, D, F) or (None,) * 3)[:3] == (down or (None,) * 3)


@pytest.mark.parametrize("hd,heads,hkv,B,H,keys,splits", [  # the sizes of test_gpu_attention_groups
    (256, 2, 1, 130, 16, 5 * 32, 1), (256, 2, 1, 130, 16, 6 * 32 - 31, 1), (128, 4, 2, 70, 9, 9 * 32 - 5, 1),
    (64, 4, 4, 40, 20, 10 * 32 - 1, 1), (256, 2, 1, 40, 16, 25 * 32 - 7, 5), (128, 2, 1, 30, 16, 70 * 32 - 3, 7),
])
def test_two_key_group_sizes(hd, heads, hkv, B, H, keys, splits):
    small = R.projection(R.GEGLU, B * H, 2 * 256, 128)[0] == R.SMALL
    got, per, two, most = R.attention(heads, hkv, hd, B, H, keys, small_gateup=small)
    assert two == 1 and got == splits <= most and got * per >= (keys + 31) // 32


@pytest.mark.parametrize("B,H,prefix,small,other", [  # eight query heads of 256 on one KV head
    (4, 60, 816, 7, 6), (5, 48, 900, 8, 6), (6, 42, 700, 6, 5),  # all that there may be, up to eight
    (5, 42, 700, 8, 6), (8, 24, 300, 6, 3),
    (3, 64, 1000, 7, 7), (7, 28, 1000, 7, 7),                    # nine: CUs left to the read-ahead
    (3, 32, 640, 11, 6), (3, 37, 501, 9, 5),                     # one chunk on 5/8 of the CUs
    (2, 56, 700, 6, 6), (2, 60, 816, 7, 7), (1, 50, 816, 14, 14),
])
def test_key_splits_go_by_what_gateup_gains(B, H, prefix, small, other):
    """CUs are left to the weight read-ahead only where gate/up gains by it."""
    for flag, want in ((True, small), (False, other)):
        splits, per, _, most = R.attention(8, 1, 256, B, H, prefix + H, small_gateup=flag)
        assert splits == want <= most and splits * per >= (prefix + H + 31) // 32


@pytest.mark.parametrize("H,keys,whole", [(28, 1028, True), (17, 1027, False), (24, 1024, False), (48, 864, False),
                                          (49, 865, True), (50, 866, True)])
def test_merge_reads_ahead_for_as_long_as_it_runs(H, keys, whole):
    """Batch 1 of the 1024-wide expert: down and the next layer's QKV are 13.6 MB.
    Past 16 splits the merge runs longer and reads twice as much meanwhile."""
    splits = R.attention(8, 1, 256, 1, H, keys, small_gateup=True)[0]
    got = R.merge_read_ahead(8 * H, 256, splits)
    assert (splits > 16) == (keys > 1024) and got == (8 * H + 63) // 64 * 4 * 1024 * (960 if splits > 16 else 480)
    assert (got >= 2 * 1024 * (4096 + 2560)) == whole


@pytest.mark.parametrize("n_cu", [32, 64, 128, 256])
def test_key_splits_fit_the_workspace(n_cu):
    for heads, hkv, hd in ((8, 1, 256), (12, 2, 128), (4, 4, 64)):
        for B in (1, 2, 3, 5, 8, 17, 64):
            for H in (1, 10, 37, 64):
                for keys in range(H, 1200, 53):
                    for flag in (False, True):
                        splits, per, _, most = R.attention(heads, hkv, hd, B, H, keys, n_cu, flag)
                        assert 1 <= splits <= most <= 32 and (splits - 1) * per < (keys + 31) // 32 <= splits * per


@pytest.mark.parametrize("n_cu", [32, 64, 128, 256])
def test_unmapped_modulations_stay_on_the_small_kernel(n_cu):
    """Only the small-M kernel takes a residual projection's gate by token row
    (mod_row null) or forms the next operand from a modulation: the ring and
    register-streamed kernels read mod_row for every gated row.  On a chip cut
    into partitions a few rows fill half the CUs."""
    for d in range(32, 2049, 32):
        for rows in (*range(1, 256, 9), 63, 64, 65, 128, 129, 192, 193, 255, 256, 1400, 3200):
            for K in (d, 2048, 4096):
                for scale_next in (False, True):
                    r = R.projection(R.RESID, rows, d, K, n_cu, gate=True, scale_next=scale_next)
                    assert r[0] == R.SMALL, (n_cu, d, rows, K, r)


@pytest.mark.parametrize("n_env,hkv,n_blk,launches", [
    (64, 1, 27, 1), (64, 64, 4095, 1), (64, 64, 4096, 2), (512, 128, 2048, 9), (3, 4096, 4096, 6), (1, 1, 1 << 24, 2),
])
def test_prefix_pack_launches_cover_any_size(n_env, hkv, n_blk, launches):
    """Every (environment, block) once, each launch below 2^24 workgroups."""
    got = R.pack_launches(n_env, hkv, n_blk)
    assert len(got) == launches
    assert all(e * hkv * b < 1 << 24 for _, e, _, b in got)
    assert sum(e * b for _, e, _, b in got) == n_env * n_blk
    spans = sorted((e0, q0) for e0, _, q0, _ in got)
    assert len(set(spans)) == launches and max(e0 + e for e0, e, _, _ in got) == n_env
    assert max(q0 + b for _, _, q0, b in got) == n_blk


@pytest.mark.parametrize("n_cu", [32, 64, 128, 256])
def test_residual_routes_are_the_compiled_ones(n_cu):
    """Every residual route has its kernel, and every kernel a route."""
    seen = set()
    for d in (256, 288, 384, 1024, 1536, 1920, 2048):
        for rows in (*range(1, 400, 7), *range(400, 6400, 31)):
            for K in (32, 1024, 1536, 2048, 4096, 6144):
                seen.add(R.projection(R.RESID, rows, d, K, n_cu)[:3])
    ring = {(R.RING, 64, 64), (R.RING, 128, 96), (R.RING, 128, 128)}
    assert seen == ring | {(R.SMALL, 0, 0), (R.STREAMED, 128, 96)}


@pytest.mark.parametrize("width,rows,o,down", [  # the sizes of the split-K cases of test_gpu_edges
    (1024, 1600, (64, 64, 1), (128, 128, 2)), (1024, 1100, (64, 64, 1), (128, 128, 3)),
    (1536, 1024, (64, 64, 1), (128, 96, 2)), (1536, 1000, (64, 64, 1), (128, 96, 2)),
    (1024, 3200, (128, 128, 1), (128, 128, 2)), (1536, 2048, (128, 96, 1), (128, 96, 2)),
])
def test_split_k_sizes(width, rows, o, down):
    q_dim, F = (2048, 4096) if width == 1024 else (1536, 6144)
    for K, want in ((width, o), (q_dim, o), (F, down)):  # time MLP out, O, down
        r = R.projection(R.RESID, rows, width, K)
        assert r[0] == R.RING and r[1:4] == want


@pytest.mark.parametrize("d,heads,hd,F,rows,time_mlp,o,down", [  # the sizes of test_gpu_adarms_batched.WIDE
    (1024, 8, 256, 4096, 3200, (R.STREAMED, 128, 128, 1, 0), (R.RING, 128, 128, 1, 0), (R.RING, 128, 128, 2, 0)),
    (1536, 12, 128, 6144, 1408, (R.STREAMED, 128, 128, 1, 1), (R.STREAMED, 128, 96, 1, 1), (R.RING, 128, 96, 2, 0)),
    (1536, 4, 64, 2048, 1397, (R.STREAMED, 128, 128, 1, 1), (R.STREAMED, 128, 96, 1, 0), (R.STREAMED, 128, 96, 1, 1)),
    (1536, 12, 128, 6144, 2048, (R.STREAMED, 128, 128, 1, 1), (R.RING, 128, 96, 1, 0), (R.RING, 128, 96, 2, 0)),
])
def test_batched_adaptive_norm_sizes(d, heads, hd, F, rows, time_mlp, o, down):
    assert R.projection(R.SILU, rows, d, d) == time_mlp
    assert R.projection(R.MOD, rows, 14 * d, d)[0] == R.STREAMED
    assert R.projection(R.RESID, rows, d, heads * hd, gate=True, mod_row=True) == o
    assert R.projection(R.RESID, rows, d, F, gate=True, mod_row=True) == down


def test_pi05_batched_sizes():
    """The 8- and 24-environment cases of test_gpu_adarms."""
    for rows, o, down in ((400, (R.SMALL, 0, 0, 1), (R.RING, 64, 64, 4)), (1200, (R.RING, 64, 64, 1), (R.RING, 128, 128, 3))):
        assert R.projection(R.SILU, rows, 1024, 1024)[0] == R.SMALL
        assert R.projection(R.MOD, rows, 110 * 1024, 1024)[0] == R.STREAMED
        assert R.projection(R.RESID, rows, 1024, 2048, gate=True, mod_row=True)[:4] == o
        assert R.projection(R.RESID, rows, 1024, 4096, gate=True, mod_row=True)[:4] == down


def test_split_short_k_sizes():
    """A width without 64 x 64 tiles: the short K splits too (test_gpu_ring_tiles)."""
    for K in (288, 1024):
        assert R.projection(R.RESID, 3750, 288, K)[:4] == ((R.RING, 128, 96, 2) if K == 1024 else (R.SMALL, 0, 0, 1))


@pytest.mark.parametrize("d,F,at_256", [(256, 1024, False), (512, 2048, False), (768, 3072, True), (1024, 4096, True),
                                        (1536, 6144, True)])
def test_adaptive_norms_by_class(d, F, at_256):
    """256 rows go by class where gate/up then takes the ring; by token the small-M
    kernel has its last whole row groups, and a schedule conditions once."""
    assert [R.ada_by_class(M, d, F) for M in (1, 255, 256, 257, 3200)] == [False, False, at_256, True, True]
    assert (R.projection(R.GEGLU, 256, 2 * F, d)[0] == R.RING) == at_256


def test_adaptive_norm_bound_sizes():
    """The sizes of test_gpu_adarms_batched.test_schedule_at_the_bound."""
    assert not R.ada_by_class(256, 256, 1024) and R.ada_by_class(256, 768, 3072)
    assert R.projection(R.MOD, 256, 26 * 256, 256)[0] == R.STREAMED  # by token: the first norm's operand formed there
    assert R.projection(R.RESID, 256, 256, 1024, gate=True, scale_next=True)[0] == R.SMALL
