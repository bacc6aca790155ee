"""GPU parity of the decode call at the borders of its split plan (number of (sequence, KV head)
pairs and of visited halves), where the output comes from the split kernel itself (one split), and
where some of the workgroup's four waves have no keys; against the fp64 CPU oracle.
"""
import math

import numpy as np
import pytest
import torch

from oracle import swaa_decode_oracle
from paper_2512_10411_amd import binding
from paper_2512_10411_amd.inputs import make_qkv
from gpu_util import assert_parity, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,G,Nq,Nk,W,S", [
    (1, 1, 4, 1, 512, 10**9, 0),      # 16 halves: the longest that one workgroup takes alone
    (1, 1, 4, 1, 513, 10**9, 0),      # 17: several splits
    (1, 2, 4, 1, 97, 10**9, 0),       # four halves and one key: the last wave has none
    (127, 1, 1, 1, 1100, 10**9, 4),   # 127 pairs: two splits
    (1, 1, 4, 1, 6177, 10**9, 4),     # 194 halves: the most splits a pair gets
    (128, 1, 2, 1, 3072, 10**9, 4),   # 128 pairs, 96 halves: one split
    (128, 1, 2, 1, 3073, 10**9, 4),   # ... and 97
    (257, 1, 1, 1, 3100, 10**9, 0),   # more than 256 pairs: four
    (513, 1, 1, 1, 3100, 10**9, 0),   # more than the workgroups that run at once: four
    (64, 2, 4, 9, 600, 10**9, 4),     # two column tiles, one split
    (3, 2, 5, 13, 2000, 900, 40),     # three column tiles (one workgroup with a single one), many splits, window + sinks
    (16, 8, 5, 8, 300, 10**9, 4),     # 128 pairs of column tiles: a workgroup for each tile
    (64, 2, 3, 21, 300, 100, 4),      # ... with window; the second tile has 31 columns
    (86, 3, 5, 8, 300, 10**9, 0),     # 258 pairs: a workgroup for each tile again
    (65, 2, 5, 16, 300, 10**9, 0),    # three tiles, 260 pairs
    (257, 1, 4, 1, 2048, 10**9, 4),   # 257 pairs of one tile, 64 halves: four splits
    (257, 1, 4, 1, 2016, 10**9, 4),   # ... and 63: one
    (321, 1, 4, 1, 2048, 10**9, 4),   # 321 pairs: one
    (42, 3, 5, 8, 2000, 10**9, 4),    # 126 pairs of column tiles: two tiles a workgroup, two splits
])
def test_borders_of_the_split_plan(B, Hkv, G, Nq, Nk, W, S):
    tag = f"decode B{B} Hkv{Hkv} G{G} Nq{Nq} Nk{Nk} W{W} S{S}"
    print(f"[case] {tag}", flush=True)
    q, k, v = make_qkv(B, Hkv * G, Hkv, Nk, 128, seed=97000 + B + Nk, n_query=Nq)
    out, lse = binding.swaa_attn_decode(to_device(q), to_device(k), to_device(v), W, S)
    torch.cuda.synchronize()
    ro, rl = swaa_decode_oracle(q, k, v, W, S, 1 / math.sqrt(128))
    assert_parity(out, lse, ro, rl, tag=tag)


def test_sequences_of_one_split_beside_long_ones():
    # per-sequence lengths: short sequences leave the split kernel finished, long ones go through the merge
    lens = [1, 32, 33, 129, 500, 9000, 17, 3000]
    host = [make_qkv(1, 8, 2, n, 128, 97900 + i, n_query=1) for i, n in enumerate(lens)]
    q = torch.cat([to_device(h[0]) for h in host])
    k = torch.zeros((len(lens), 2, max(lens), 128), dtype=torch.bfloat16, device="cuda")
    v = torch.zeros_like(k)
    for b, (h, n) in enumerate(zip(host, lens)):
        k[b, :, :n], v[b, :, :n] = to_device(h[1])[0], to_device(h[2])[0]
    sl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    for W in (10**9, 300):
        out, lse = binding.swaa_attn_decode_ex(q, k, v, W, 4, seq_lens=sl)
        torch.cuda.synchronize()
        for b, h in enumerate(host):
            ro, rl = swaa_decode_oracle(*h, W, 4, 1 / math.sqrt(128))
            assert_parity(out[b:b + 1], lse[b:b + 1], ro, rl, tag=f"seq {b} of {lens[b]} W{W}")


def test_several_splits_of_single_column_tiles_and_the_static_array():
    # 264 pairs of column tiles on 4.1k tokens: four splits in a workspace, fewer where the library's own array must do
    B, G, Nq, Nk = 264, 5, 8, 4100
    assert binding.swaa_attn_decode_workspace_bytes(B, G, 1, Nq, Nk, 128, Nk, 4) > binding.SWAA_DECODE_STATIC_SCRATCH_BYTES
    q, k, v = make_qkv(B, G, 1, Nk, 128, seed=97800, n_query=Nq)
    qd, kd, vd = to_device(q), to_device(k), to_device(v)
    out, lse = binding.swaa_attn_decode(qd, kd, vd, Nk, 4)
    out1, lse1 = torch.full_like(out, float("nan")), torch.full_like(lse, float("nan"))
    binding.swaa_attn_decode_static(qd, kd, vd, out1, lse1, Nk, 4)
    torch.cuda.synchronize()
    some = slice(0, B, 29)
    ro, rl = swaa_decode_oracle(q[some], k[some], v[some], Nk, 4, 1 / math.sqrt(128))
    assert_parity(out[some], lse[some], ro, rl, tag="splits in a workspace")
    assert_parity(out1[some], lse1[some], ro, rl, tag="static array")


def test_several_splits_of_two_column_tiles_where_the_last_round_is_nearly_empty():
    B, G, Nq, Nk = 17, 4, 512, 12300  # 17 x 32 pairs of column tiles
    q, k, v = make_qkv(B, G, 1, Nk, 128, seed=97810, n_query=Nq)
    out, lse = binding.swaa_attn_decode(to_device(q), to_device(k), to_device(v), Nk, 4)
    torch.cuda.synchronize()
    for b in (0, B - 1):
        one = slice(b, b + 1)
        ro, rl = swaa_decode_oracle(q[one], k[one], v[one], Nk, 4, 1 / math.sqrt(128))
        assert_parity(out[one], lse[one], ro, rl, tag=f"sequence {b}")


@pytest.mark.parametrize("first,last", [(2560, 3072), (5, 6), (0, 8000)])  # splits of 256 keys: two whole ones
def test_keys_that_are_no_numbers_show_in_the_rows_that_see_them(first, last):
    # whole splits of NaN among them: the merge must not take those for splits without keys
    q, k, v = make_qkv(1, 4, 1, 8000, 128, seed=97820, n_query=1)
    k[:, :, first:last, 7] = np.uint16(0x7FC0)
    out, lse = binding.swaa_attn_decode(to_device(q), to_device(k), to_device(v), 8000, 4)
    seen = binding.swaa_attn_decode_ex(to_device(q), to_device(k), to_device(v), 8000, 4,
                                       seq_lens=torch.tensor([8000], dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    for o, l in ((out, lse), seen):
        assert not torch.isfinite(o.float()).any() and not torch.isfinite(l).any()
