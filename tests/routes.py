"""The library's dispatch rules (csrc/routes.h) on the CPU, for any CU count:
the header is compiled as it stands with the host compiler."""
from __future__ import annotations

import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SILU, RESID, GEGLU, QKV, MOD = 0, 1, 3, 4, 5
SMALL, STREAMED, RING = 0, 1, 2

SRC = r"""
#include "%s/paper_2609_37772_amd/csrc/routes.h"
using namespace uad;
extern "C" void projection(const int *a, int *out) {  // n_cu epi M N K q_dim second gate mod_row scale_next
  Proj p{a[0], a[1], a[2], a[3], a[4], a[5], a[6] != 0, a[7] != 0, a[8] != 0, a[9] != 0,
         (size_t)2 * a[0] * 128 * 128 * 4, a[0]};  // the workspace that a context has
  const ProjRoute r = route_projection(p);
  out[0] = r.kernel; out[1] = r.rows; out[2] = r.cols; out[3] = r.kx; out[4] = r.halves;
}
extern "C" void attention(const int *a, int *out) {  // n_cu group n_kv_heads head_dim B H keys small_gateup
  AttnSizes s{a[0], a[1], a[2], a[3], a[4], a[5], (a[6] + 31) / 32, a[7] != 0};
  const int nb = attn_chunk_blocks(s.head_dim);
  out[0] = attn_splits(s, &out[1]);
  const int groups = s.B * s.n_kv_heads * out[0];
  out[2] = attn_two_groups(s.n_cu, groups, s.qblocks(), out[1], nb);
  out[3] = attn_splits_max(s);
}
extern "C" long merge_bytes(int rows_pad, int head_dim, int splits) { return merge_read_ahead(rows_pad, head_dim, splits); }
extern "C" int by_class(int n_cu, int M, int d, int F) { return ada_by_class(n_cu, M, d, F); }
extern "C" int pack_launches(const int *a, int *out) {  // n_env n_kv_heads n_blk -> (env envs blk blks)*, how many
  int n = 0;
  for_pack_launches(a[0], a[1], a[2], [&](int e, int ne, int q, int nq) {
    const int v[4] = {e, ne, q, nq};
    std::copy(v, v + 4, out + 4 * n);
    return (int)(++n == 64);
  });
  return n;
}
"""


@functools.lru_cache(None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "routes.cpp"), os.path.join(d, "routes.so")
        with open(src, "w") as fh:
            fh.write(SRC % ROOT)
        subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", src, "-o", so], check=True)
        return ctypes.CDLL(so)


def _call(fn, args, n_out):
    a, out = (ctypes.c_int * len(args))(*[int(v) for v in args]), (ctypes.c_int * n_out)()
    getattr(_lib(), fn)(a, out)
    return tuple(out)


def projection(epi, M, N, K, n_cu=256, q_dim=0, second=False, gate=False, mod_row=False, scale_next=False):
    """(kernel, tile rows, tile columns, split over K, k-halves)."""
    return _call("projection", (n_cu, epi, M, N, K, q_dim, second, gate, mod_row, scale_next), 5)


def attention(heads, n_kv_heads, head_dim, B, H, keys, n_cu=256, small_gateup=False):
    """(key splits, 32-key blocks of each, two key groups, most splits)."""
    return _call("attention", (n_cu, heads // n_kv_heads, n_kv_heads, head_dim, B, H, keys, small_gateup), 4)


def merge_read_ahead(rows, head_dim, splits):
    """Bytes that the split merge may read ahead (below 256 token rows)."""
    fn = _lib().merge_bytes
    fn.restype = ctypes.c_long
    return fn((rows + 63) // 64 * 64, head_dim, splits)


def ada_by_class(M, d, F, n_cu=256):
    """Whether the adaptive norms of a step of M rows go by flow-time class."""
    return bool(_lib().by_class(n_cu, M, d, F))


def pack_launches(n_env, n_kv_heads, n_blk):
    """The launches of a prefix repacking: (first environment, environments, first block, blocks)."""
    a, out = (ctypes.c_int * 3)(n_env, n_kv_heads, n_blk), (ctypes.c_int * 256)()
    n = _lib().pack_launches(a, out)
    return [tuple(out[4 * i:4 * i + 4]) for i in range(n)]
